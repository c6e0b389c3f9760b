"""Symmetric diagonals at their edges: operands with infinities, and operators
whose entries above the diagonal have no mirror image, or a zero one, and a
layout taken away again."""
import numpy as np
import pytest

from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev
from tests.test_gpu_slices import _entrywise
from tests.test_gpu_sym_diagonals import CASES

pytestmark = pytest.mark.gpu

amg = pytest.importorskip("paper_1403_1649_amd")


@pytest.mark.parametrize("sched", ["contiguous", "sweep"])
@pytest.mark.parametrize("name", CASES)
def test_infinity_reaches_only_the_rows_that_meet_it(name, sched, monkeypatch):
    """The rows whose entries meet an infinite x_j become infinite, no others:
    an offset that a row does not have (past the grid's edge, past either end)
    adds nothing."""
    make, dim = CASES[name]
    A = make()
    monkeypatch.setenv("AMG_TUNE_FORCE", "symdia")
    monkeypatch.setenv("AMG_TUNE_SCHEDULE", sched)
    h = amg.setup(*to_dev(A), amg.Options(dim=dim))
    assert h.level_format(0)[0] == 5
    S = A.to_scipy().tocsr()
    rng = np.random.default_rng(5)
    for at in ([0, A.n - 1], [255, A.n - 300], list(rng.integers(1000, A.n - 1000, 1))):
        x = P.exact_solution(A.n, 7)
        x[at] = np.inf
        y = h.level_spmv(0, dev_vec(x)).cpu().numpy()
        ref = S @ x
        inf = ~np.isfinite(ref)
        assert inf.sum() == np.unique(S[:, at].tocoo().row).size
        assert np.array_equal(~np.isfinite(y), inf) and np.array_equal(y[inf], ref[inf])
        # both sides sum at most five to nine products: each within (count - 1) u of the exact row sum
        rowlen = np.diff(S.indptr).max()
        bound = 2.5e-16 * rowlen * (abs(S) @ np.where(np.isfinite(x), np.abs(x), 0.0))
        assert np.all(np.abs(y[~inf] - ref[~inf]) <= bound[~inf])
    h.close()


@pytest.mark.parametrize("krylov", ["fcg", "fgmres"])
def test_entries_above_without_a_mirror_image(krylov, monkeypatch):
    """Identity rows on the last grid line, the columns not eliminated.  Stored
    zeros in those rows: not symmetric, laid out otherwise.  No entries there:
    the pattern is refused."""
    B = P.poisson2d(300).to_scipy().tocsr()
    row = np.repeat(np.arange(B.shape[0]), np.diff(B.indptr))
    last = row >= B.shape[0] - 300
    B.data[last] = np.where(B.indices[last] == row[last], 1.0, 0.0)
    A = P.CSR(B.indptr, B.indices, B.data)
    monkeypatch.setenv("AMG_TUNE_FORCE", "symdia")
    h = amg.setup(*to_dev(A), amg.Options(dim=2, krylov=krylov))
    assert h.level_format(0)[0] != 5
    x = P.exact_solution(A.n, 9)
    y = h.level_spmv(0, dev_vec(x)).cpu().numpy()
    assert np.all(np.abs(y - B @ x) <= 2.5e-16 * 5 * (abs(B) @ np.abs(x)))
    h.close()
    B.eliminate_zeros()
    with pytest.raises(amg.AmgError, match="not structurally symmetric"):
        amg.setup(*to_dev(P.CSR(B.indptr, B.indices, B.data)), amg.Options(dim=2, krylov=krylov))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_resetup_of_an_early_layout_to_nonsymmetric_values(precision):
    """The second setup of a shape lays level 0 out before its Arnoldi products
    and builds no sliced ELL; a re-setup then takes the layout away, and later
    values that are symmetric again find the sliced diagonals."""
    A = P.poisson3d(73)
    b = P.rhs(A, P.exact_solution(A.n, 3))
    dev = to_dev(A)
    amg.setup(*dev, amg.Options(dim=3, precision=precision)).close()
    h = amg.setup(*dev, amg.Options(dim=3, precision=precision))
    assert h.level_format(0)[0] == 5
    v = np.array(A.val)
    k = int(A.row_ptr[A.n // 2])
    v[k] = np.nextafter(v[k], 0.0)   # one rounding off: still solvable by flexible CG
    for val in (v, A.val):
        M = P.CSR(A.row_ptr, A.col, val)
        h.resetup(dev_vec(val))
        assert h.level_format(0)[0] == 3
        _entrywise(h, 0, 101)
        x, _, rel = amg.solve(h, dev_vec(b), 1e-8)
        assert rel <= 1e-8
        assert np.linalg.norm(b - M.to_scipy() @ x.cpu().numpy()) <= 1.01e-8 * np.linalg.norm(b)
    h.close()
