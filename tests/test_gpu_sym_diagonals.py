"""Symmetric diagonals: a structured level whose operator equals its transpose
bit for bit stores the main diagonal and those above it, and reads the ones
below at shifted rows.  Products entry by entry and solves on five-, seven- and
nine-point grids (ragged last slices, every schedule), and the ways out: a
nonsymmetric operator of a shape tuned as symmetric, and a re-setup to values
that are not symmetric any more."""
import numpy as np
import pytest
import scipy.sparse as sp

from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev
from tests.test_gpu_post_operator import _csr
from tests.test_gpu_slices import _entrywise

pytestmark = pytest.mark.gpu

amg = pytest.importorskip("paper_1403_1649_amd")


def _nine_point(n):
    one = sp.diags([np.ones(n - 1), np.ones(n), np.ones(n - 1)], [-1, 0, 1])
    return _csr(9.0 * sp.identity(n * n) - sp.kron(one, one))


CASES = {
    "five": (lambda: P.poisson2d(261, 257), 2),
    "seven": (lambda: P.hetero3d(43, seed=4), 3),     # 79,507 rows: 19 in the last slice
    "nine": (lambda: _nine_point(263), 2),
}


def _check(h, A, b):
    x, it, rel = amg.solve(h, dev_vec(b), 1e-8)
    assert rel <= 1e-8
    assert np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) <= 1.01e-8 * np.linalg.norm(b)
    return it


@pytest.mark.parametrize("sched", ["contiguous", "sweep"])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("name", CASES)
def test_products_and_solve(name, precision, sched, monkeypatch):
    make, dim = CASES[name]
    A = make()
    b = P.rhs(A, P.exact_solution(A.n, 3))
    print(f"symmetric diagonals: {name} {precision} {sched}", flush=True)
    h0 = amg.setup(*to_dev(A), amg.Options(dim=dim, precision=precision))
    it0 = _check(h0, A, b)
    h0.close()
    monkeypatch.setenv("AMG_TUNE_FORCE", "symdia")
    monkeypatch.setenv("AMG_TUNE_SCHEDULE", sched)
    h = amg.setup(*to_dev(A), amg.Options(dim=dim, precision=precision))
    assert h.level_format(0, "fp64")[:2] == (5, 1)
    _entrywise(h, 0, 81)
    assert abs(_check(h, A, b) - it0) <= 1
    h.resetup(to_dev(A)[2] * 2.0)
    assert h.level_format(0, "fp64")[:2] == (5, 1)
    _entrywise(h, 0, 82)
    A2 = P.CSR(A.row_ptr, A.col, 2.0 * np.asarray(A.val))
    assert abs(_check(h, A2, b) - it0) <= 1
    h.close()


def test_plane_schedule(monkeypatch):
    A = P.poisson3d(64)
    monkeypatch.setenv("AMG_TUNE_FORCE", "symdia")
    monkeypatch.setenv("AMG_TUNE_SCHEDULE", "plane")
    h = amg.setup(*to_dev(A), amg.Options(dim=3))
    assert h.level_format(0)[:2] == (5, 1)
    _entrywise(h, 0, 83)
    _check(h, A, P.rhs(A, P.exact_solution(A.n, 3)))
    h.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_resetup_to_nonsymmetric_values(precision, monkeypatch):
    """One value off its mirror image by a rounding: still solvable by FCG, but
    not in symmetric diagonals."""
    A = P.hetero3d(43, seed=4)
    b = P.rhs(A, P.exact_solution(A.n, 3))
    monkeypatch.setenv("AMG_TUNE_FORCE", "symdia")
    h = amg.setup(*to_dev(A), amg.Options(dim=3, precision=precision))
    assert h.level_format(0, "fp64")[0] == 5
    v = np.array(A.val)
    row = A.n // 2
    k = int(A.row_ptr[row])
    assert A.col[k] < row
    v[k] = np.nextafter(v[k], 0.0)
    A2 = P.CSR(A.row_ptr, A.col, v)
    h.resetup(to_dev(A2)[2])
    assert h.level_format(0, "fp64")[0] == 3
    _entrywise(h, 0, 84)
    _check(h, A2, b)
    h.close()


def test_nonsymmetric_operator_of_a_tuned_shape():
    """The decision kept for a shape does not depend on the values: a matrix of
    the same pattern that is not symmetric is laid out otherwise."""
    S = P.poisson2d(263, 259)
    b = P.rhs(S, P.exact_solution(S.n, 3))
    h = amg.setup(*to_dev(S), amg.Options(dim=2))
    it0 = _check(h, S, b)
    h.close()
    v = np.array(S.val)
    row = np.repeat(np.arange(S.n), np.diff(S.row_ptr))
    v[(np.asarray(S.col) == row + 1)] *= 0.5
    A = P.CSR(S.row_ptr, S.col, v)
    bA = P.rhs(A, P.exact_solution(A.n, 3))
    h = amg.setup(*to_dev(A), amg.Options(dim=2, krylov="fgmres"))
    assert h.level_format(0)[0] != 5
    _entrywise(h, 0, 85)
    _check(h, A, bA)
    h.close()
    h = amg.setup(*to_dev(S), amg.Options(dim=2))
    assert abs(_check(h, S, b) - it0) <= 1
    h.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("make", [lambda: P.poisson3d(71), lambda: P.poisson2d(700), lambda: _nine_point(267)],
                         ids=["seven", "five", "nine"])
def test_second_setup_of_a_tuned_shape(make, precision):
    """A setup that finds its shape's decision lays level 0 out before the
    Arnoldi products and without the sliced ELL: the same weights bit for bit
    (the same rows per thread and block) and the same solve."""
    A = make()
    b = P.rhs(A, P.exact_solution(A.n, 3))
    got = []
    for _ in range(2):
        h = amg.setup(*to_dev(A), amg.Options(dim=3 if A.n == 71 ** 3 else 2, precision=precision))
        got.append((h.level_info(0)["omega"], h.level_format(0, "fp64")[0], _check(h, A, b)))
        _entrywise(h, 0, 86)
        h.resetup(to_dev(A)[2])
        assert abs(_check(h, A, b) - got[-1][2]) <= 1
        h.close()
    assert got[0] == got[1]
