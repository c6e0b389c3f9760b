"""Batched cycles by the post-smoothing operator T_k: systems whose rows fill a
64-row group of T beyond what one turn of the streaming kernel holds, rows of
many aggregates, a row too long for T on one system (its level then
post-smooths with A_k), and more systems than the per-system reductions have
blocks.  Each system converges as it does alone (iterations within one, x to
1e-6, the solve's stopping tolerance times its margin for a differing count)."""
import numpy as np
import pytest

from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev
from tests.test_gpu_post_operator import _arrow, _stencil27

pytestmark = pytest.mark.gpu

amg = pytest.importorskip("paper_1403_1649_amd")

CASES = {
    "stencil27": lambda: [P.poisson3d(9), _stencil27(23), P.hetero3d(14, seed=4), _stencil27(15)],
    "arrow_500": lambda: [P.poisson2d(40), _arrow(60, 50, 500), P.poisson2d(31)],
    "arrow_600": lambda: [P.poisson2d(40), _arrow(60, 50, 600), P.poisson2d(31)],
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", CASES)
def test_systems_match_single_solves(name, precision):
    mats = CASES[name]()
    Abd, off = P.block_diag(mats)
    print(f"batch: {name} {precision} n={Abd.n}", flush=True)
    b = P.rhs(Abd, P.exact_solution(Abd.n, 2))
    h = amg.setup_batched(*to_dev(Abd), off, amg.Options(dim=3, precision=precision))
    x = amg.solve(h, dev_vec(b), 1e-8)[0].cpu().numpy()
    its, rels = h.batch_results()
    for q, m in enumerate(mats):
        lo, hi = off[q], off[q + 1]
        hs = amg.setup(*to_dev(m), amg.Options(dim=3, precision=precision))
        x1, it1, _ = amg.solve(hs, dev_vec(b[lo:hi]), 1e-8)
        assert rels[q] <= 1e-8 and abs(int(its[q]) - it1) <= 1, (q, its[q], it1)
        assert np.linalg.norm(b[lo:hi] - m.to_scipy() @ x[lo:hi]) <= 1.01e-8 * np.linalg.norm(b[lo:hi])
        assert np.linalg.norm(x[lo:hi] - x1.cpu().numpy()) <= 1e-6 * np.linalg.norm(x1.cpu().numpy())
        hs.close()
    h.close()


@pytest.mark.parametrize("nsys", [2047, 2049])
def test_more_systems_than_reduction_blocks(nsys):
    mats = [P.poisson2d(1 + q % 3, 1 + q % 2) for q in range(nsys - 1)] + [P.poisson2d(33)]
    Abd, off = P.block_diag(mats)
    b = P.rhs(Abd, P.exact_solution(Abd.n, 2))
    h = amg.setup_batched(*to_dev(Abd), off, amg.Options(dim=2))
    x = amg.solve(h, dev_vec(b), 1e-8)[0].cpu().numpy()
    its, rels = h.batch_results()
    r = b - Abd.to_scipy() @ x
    for q in range(nsys):
        lo, hi = off[q], off[q + 1]
        assert rels[q] <= 1e-8 and np.linalg.norm(r[lo:hi]) <= 1.01e-8 * np.linalg.norm(b[lo:hi]), q
        assert its[q] == 1 or q == nsys - 1   # a system of one level: its dense inverse
    h.close()
