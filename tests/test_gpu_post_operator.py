"""The post-smoothing operator T_k = (I - W A_k) P_k: damped-Jacobi cycles
take the corrected and post-smoothed iterate as y + T_k e instead of by a
second product with A_k.  Solves against the oracle (whose cycle applies A_k
twice) on matrices that reach each kernel: streamed rows whose 64-row groups
hold up to 256, 320 or 512 entries, rows of more than eight distinct
aggregates and of more entries than a wave takes at a time, small levels (a
wave per row), and a level with a row too long for T, which post-smooths with
A_k as before."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import amg_oracle as O
from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1403_1649_amd")


def _csr(S):
    S = S.tocsr()
    S.sort_indices()
    return P.CSR(S.indptr, S.indices, S.data)


def _stencil27(n):
    """27-point Laplacian on n^3 (diagonal 26, every neighbour -1)."""
    one = sp.diags([np.ones(n - 1), np.ones(n), np.ones(n - 1)], [-1, 0, 1])
    return _csr(27.0 * sp.identity(n ** 3) - sp.kron(sp.kron(one, one), one))


def _arrow(nx, ny, m):
    """2-D Poisson with unknown 0 also coupled to the last m unknowns."""
    S = P.poisson2d(nx, ny).to_scipy().tocoo()
    n = nx * ny
    j = np.arange(n - m, n)
    w = np.full(m, 1e-3)
    d = np.zeros(n)
    d[j] += w
    d[0] += w.sum()
    z = np.zeros(m, dtype=int)
    return _csr(S + sp.coo_matrix((np.concatenate([-w, -w]), (np.concatenate([z, j]), np.concatenate([j, z]))),
                                  shape=(n, n)) + sp.diags(d))


CASES = {
    "poisson2d_streamed": (lambda: P.poisson2d(263, 257), 2),        # five entries a row, ragged last group
    "hetero3d_streamed": (lambda: P.hetero3d(41, seed=4), 3),        # seven
    "stencil27_streamed": (lambda: _stencil27(41), 3),               # 27: several turns per 64 rows
    "hetero3d_small": (lambda: P.hetero3d(17, seed=4), 3),           # every level a wave per row
    "arrow_600": (lambda: _arrow(60, 50, 600), 2),                   # a row of over 512 entries
    "arrow_500": (lambda: _arrow(60, 50, 500), 2),                   # and one just below, many aggregates
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", CASES)
def test_solve_with_post_operator_matches_oracle(name, precision):
    make, dim = CASES[name]
    A = make()
    b = P.rhs(A, P.exact_solution(A.n, 3))
    print(f"post operator: {name} {precision} n={A.n}", flush=True)
    h = amg.setup(*to_dev(A), amg.Options(dim=dim, precision=precision))
    x, it, rel = amg.solve(h, dev_vec(b), 1e-8)
    x = x.cpu().numpy()
    ref = O.solve(O.setup(A.row_ptr, A.col, A.val, O.Options.for_dim(dim)), b, 1e-8)
    assert rel <= 1e-8 and abs(it - ref.iters) <= 1, (it, ref.iters)
    assert np.linalg.norm(b - A.to_scipy() @ x) <= 1.01e-8 * np.linalg.norm(b)
    if it == ref.iters:
        assert np.linalg.norm(x - ref.x) <= 1e-6 * np.linalg.norm(ref.x)
    h.resetup(to_dev(A)[2] * 2.0)   # T follows the new values
    x2, it2, rel2 = amg.solve(h, dev_vec(b), 1e-8)
    assert rel2 <= 1e-8 and abs(it2 - it) <= 1
    assert np.linalg.norm(2.0 * x2.cpu().numpy() - x) <= 1e-6 * np.linalg.norm(x)
    h.close()
