"""Flexible GMRES: restart lengths from one step to more than the solve needs,
both precisions, the captured cycle against eager launches, and the coarsest
inverse of nonsymmetric operators, diagonally dominant (no pivoting) and not
(partial pivoting)."""
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


def _convdiff(nx, ny):
    S = P.poisson2d(nx, ny).to_scipy().tolil()
    for i in range(nx * ny):
        if i % nx:
            S[i, i - 1] -= 0.8
            S[i, i] += 0.8
    return _csr(S)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("nx, ny, restart", [(37, 33, 1), (37, 33, 5), (90, 61, 30), (90, 61, 64)])
def test_restart_lengths_match_oracle_and_eager(nx, ny, restart, precision):
    A = _convdiff(nx, ny)
    b = P.rhs(A, P.exact_solution(A.n, 2))
    kw = dict(krylov="fgmres", coarse_max=100, gmres_restart=restart)
    print(f"fgmres {nx}x{ny} m={restart} {precision}", flush=True)
    out = []
    for flags in (0, amg.binding.FLAG_NO_GRAPH):
        h = amg.setup(*to_dev(A), amg.Options(dim=2, precision=precision, flags=flags, **kw))
        x, it, rel = amg.solve(h, dev_vec(b), 1e-8)
        x2, it2, _ = amg.solve(h, dev_vec(b), 1e-8)
        assert rel <= 1e-8 and it2 == it and torch.equal(x, x2)
        out.append((it, x.cpu().numpy()))
        h.close()
    assert out[0][0] == out[1][0] and np.array_equal(out[0][1], out[1][1])
    ref = O.solve(O.setup(A.row_ptr, A.col, A.val, O.Options.for_dim(2, **kw)), b, 1e-8)
    assert abs(out[0][0] - ref.iters) <= 1, (out[0][0], ref.iters)
    assert np.linalg.norm(b - A.to_scipy() @ out[0][1]) <= 1.01e-8 * np.linalg.norm(b)


@pytest.mark.parametrize("n", [1, 31, 64, 361, 600])
@pytest.mark.parametrize("dominant", [True, False])
def test_nonsymmetric_coarse_inverse(n, dominant):
    """Single-level hierarchies: the preconditioner is the inverse itself."""
    rng = np.random.default_rng(n)
    if n == 1:
        S = sp.csr_matrix(np.array([[3.0]]))
    else:
        nx = int(np.ceil(np.sqrt(n)))
        S = _convdiff(nx, nx).to_scipy().tocsr()[:n, :n]
        if not dominant:   # off-diagonals far above the diagonal, both signs
            S = S.tocoo()
            off = S.row != S.col
            S.data[off] *= rng.uniform(-9.0, 9.0, off.sum())
    A = _csr(S)
    h = amg.setup(*to_dev(A), amg.Options(dim=2, krylov="fgmres", coarse_max=600))
    assert h.num_levels() == 1
    b = rng.standard_normal(n)
    x, it, rel = amg.solve(h, dev_vec(b), 1e-8)
    M = A.to_scipy().toarray()
    assert it <= 2 and rel <= 1e-8   # the solve's own tolerance, reached by the preconditioner alone
    xs = np.linalg.solve(M, b)
    # |x - xs| <= cond(M) times the relative residual
    assert np.linalg.norm(x.cpu().numpy() - xs) <= 1e-9 * np.linalg.cond(M) * np.linalg.norm(xs)
