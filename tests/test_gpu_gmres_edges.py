"""Flexible GMRES where its steps end early: a zero right-hand side, a basis that
closes after one step (the new vector is exactly zero), an iteration limit
inside a cycle."""
import numpy as np
import pytest
import scipy.sparse as sp

from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev
from tests.test_gpu_gmres import _convdiff, _csr

pytestmark = pytest.mark.gpu

amg = pytest.importorskip("paper_1403_1649_amd")

FLAGS = pytest.mark.parametrize("flags", [0, amg.binding.FLAG_NO_GRAPH], ids=["graphs", "eager"])
PRECISION = pytest.mark.parametrize("precision", ["fp64", "mixed"])


@FLAGS
@PRECISION
def test_zero_right_hand_side(precision, flags):
    A = _convdiff(61, 47)
    h = amg.setup(*to_dev(A), amg.Options(dim=2, krylov="fgmres", precision=precision, flags=flags, coarse_max=100))
    x, it, rel = amg.solve(h, dev_vec(np.zeros(A.n)), 1e-8)
    assert it == 0 and rel == 0.0 and not np.any(x.cpu().numpy())
    b = P.rhs(A, P.exact_solution(A.n, 2))
    x, _, rel = amg.solve(h, dev_vec(b), 1e-8)
    assert rel <= 1e-8 and np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) <= 1.01e-8 * np.linalg.norm(b)
    h.close()


@FLAGS
@PRECISION
def test_basis_closes_after_one_step(precision, flags):
    """A = 2 I and b a power of two times a unit vector: every product and dot is
    exact, so A z_0 lies in the basis and h_{1,0} is exactly zero."""
    A = _csr(2.0 * sp.identity(100))
    h = amg.setup(*to_dev(A), amg.Options(dim=2, krylov="fgmres", precision=precision, flags=flags))
    b = np.zeros(A.n)
    b[37] = 8.0
    x, it, rel = amg.solve(h, dev_vec(b), 1e-8)
    assert it == 1 and rel == 0.0 and np.array_equal(x.cpu().numpy(), 0.5 * b)
    h.close()


@FLAGS
def test_iteration_limit_inside_a_cycle(flags):
    A = _convdiff(90, 61)
    b = P.rhs(A, P.exact_solution(A.n, 2))
    rels = []
    for m in (1, 4, 7):
        h = amg.setup(*to_dev(A), amg.Options(dim=2, krylov="fgmres", max_iter=m, flags=flags, coarse_max=100))
        x, it, rel = amg.solve(h, dev_vec(b), 1e-12, allow_notconv=True)
        assert it == m
        true = np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) / np.linalg.norm(b)
        assert abs(true - rel) <= 1e-12
        rels.append(rel)
        h.close()
    assert rels[0] > rels[1] > rels[2] > 1e-12
