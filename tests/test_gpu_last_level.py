"""Small levels take pre-smoothing and restriction as S_k b with
S_k = P^T (I - A W), and the level above the coarsest its whole cycle (or the
coarse correction) as a dense operator.  Solves against the oracle, whose cycle
does each step by itself, with hierarchies cut so that the last level is
level 0, 1 or 2 and lies on either side of the sizes where the operators are
formed; an aggregate with more rows than S takes; new values and a
nonsymmetric operator."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import amg_oracle as O
from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev
from tests.test_gpu_post_operator import _csr

pytestmark = pytest.mark.gpu

amg = pytest.importorskip("paper_1403_1649_amd")


def _stars(m, leaves):
    """A path of m hubs, each with its own leaves (an aggregate of one hub and
    its leaves has leaves + 1 rows)."""
    n = m * (leaves + 1)
    h = np.arange(m) * (leaves + 1)
    i = np.concatenate([np.repeat(h, leaves), h[:-1]])
    j = np.concatenate([(h[:, None] + 1 + np.arange(leaves)).ravel(), h[1:]])
    S = sp.coo_matrix((np.full(i.size, -1.0), (i, j)), shape=(n, n))
    S = S + S.T
    return _csr(S + sp.diags(0.01 - np.asarray(S.sum(axis=1)).ravel()))


CASES = {
    "one_small": (lambda: P.poisson2d(26), 2, 2),          # level 0 last: C S dense
    "one_ragged": (lambda: P.poisson2d(41, 37), 2, 2),
    "one_wide": (lambda: P.poisson2d(70), 2, 2),           # level 0 last, C S too large
    "two_dense": (lambda: P.poisson2d(97, 101), 2, 3),     # level 1 last, about 1,400 rows
    "two_edge": (lambda: P.poisson2d(120), 2, 3),          # about 2,040
    "two_wide": (lambda: P.poisson2d(131), 2, 3),          # above 2,048: C S
    "two_neither": (lambda: P.poisson2d(260), 2, 3),       # about 9,500
    "three_3d": (lambda: P.hetero3d(33, seed=4), 3, 4),
    "stars": (lambda: _stars(30, 200), 2, 25),
}


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", CASES)
def test_small_levels_match_oracle(name, precision):
    make, dim, levels = CASES[name]
    A = make()
    b = P.rhs(A, P.exact_solution(A.n, 3))
    print(f"last level: {name} {precision} n={A.n}", flush=True)
    h = amg.setup(*to_dev(A), amg.Options(dim=dim, precision=precision, max_levels=levels, coarse_max=60))
    x, it, rel = amg.solve(h, dev_vec(b), 1e-8)
    x = x.cpu().numpy()
    o = O.Options.for_dim(dim)
    o.max_levels, o.coarse_max = levels, 60
    ref = O.solve(O.setup(A.row_ptr, A.col, A.val, o), b, 1e-8)
    assert rel <= 1e-8 and abs(it - ref.iters) <= 1, (it, ref.iters)
    assert np.linalg.norm(b - A.to_scipy() @ x) <= 1.01e-8 * np.linalg.norm(b)
    if it == ref.iters:
        assert np.linalg.norm(x - ref.x) <= 1e-6 * np.linalg.norm(ref.x)
    h.resetup(to_dev(A)[2] * 2.0)   # the operators follow the new values
    x2, it2, rel2 = amg.solve(h, dev_vec(b), 1e-8)
    assert rel2 <= 1e-8 and abs(it2 - it) <= 1
    assert np.linalg.norm(2.0 * x2.cpu().numpy() - x) <= 1e-6 * np.linalg.norm(x)
    h.close()


@pytest.mark.parametrize("side", [40, 90, 131])
def test_nonsymmetric_levels_match_oracle(side):
    S = P.poisson2d(side).to_scipy().tolil()
    n = side * side
    up = sp.diags([np.full(n - 1, 0.45), np.full(n - 1, -0.45)], [1, -1])
    mask = (abs(S) > 0).astype(float)
    A = _csr(S + mask.multiply(up))   # convection along the first axis, on the same pattern
    b = P.rhs(A, P.exact_solution(A.n, 3))
    print(f"last level: nonsymmetric {side}", flush=True)
    h = amg.setup(*to_dev(A), amg.Options(dim=2, krylov="fgmres", max_levels=3))
    x, it, rel = amg.solve(h, dev_vec(b), 1e-8)
    o = O.Options.for_dim(2)
    o.krylov, o.max_levels = "fgmres", 3
    ref = O.solve(O.setup(A.row_ptr, A.col, A.val, o), b, 1e-8)
    assert rel <= 1e-8 and abs(it - ref.iters) <= 1, (it, ref.iters)
    assert np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) <= 1.01e-8 * np.linalg.norm(b)
    h.close()
