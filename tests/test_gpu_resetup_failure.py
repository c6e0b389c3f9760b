"""A re-setup that fails half-way (values whose Arnoldi estimate is not finite)
leaves no captured sequence that reads what it released or gave up: the next
re-setup and solves are those of the values they are given."""
import numpy as np
import pytest

from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1403_1649_amd")


def _solve(h, A, b):
    x, _, rel = amg.solve(h, dev_vec(b), 1e-8)
    assert rel <= 1e-8
    assert np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) <= 1.01e-8 * np.linalg.norm(b)
    B = np.stack([b, -2.0 * b], axis=1)
    X, _, rels = amg.solve_multi(h, dev_vec(B), 1e-8)
    assert np.all(rels <= 1e-8)
    assert np.linalg.norm(B - A.to_scipy() @ X.cpu().numpy()) <= 1.01e-8 * np.linalg.norm(B)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("fmt, borrow", [("symdia", False), ("csr", True)], ids=["released layout", "borrowed values"])
def test_failed_resetup(fmt, borrow, precision, monkeypatch):
    A = P.hetero3d(43, seed=4)
    A2 = P.hetero3d(43, seed=5)
    b, b2 = (P.rhs(M, P.exact_solution(M.n, 3)) for M in (A, A2))
    # not symmetric any more, and an entry of D^-1 A overflows
    bad = np.array(A.val)
    row = A.n // 2
    s, e = int(A.row_ptr[row]), int(A.row_ptr[row + 1])
    bad[s] = -1e300
    bad[s + int(np.searchsorted(A.col[s:e], row))] = 1e-300
    monkeypatch.setenv("AMG_TUNE_FORCE", fmt)
    print(f"failed re-setup: {fmt} borrow={borrow} {precision}", flush=True)
    dev = to_dev(A)
    h = amg.setup(*dev, amg.Options(dim=3, precision=precision, flags=amg.binding.FLAG_BORROW_A if borrow else 0))
    assert h.level_format(0, "fp64")[0] == (5 if fmt == "symdia" else 0)
    _solve(h, A, b)
    v = dev_vec(bad)
    with pytest.raises(amg.AmgError):
        h.resetup(v)
    v.copy_(dev_vec(A2.val))   # the same address as the call that failed
    h.resetup(v)
    _solve(h, A2, b2)
    h.resetup(dev[2])
    _solve(h, A, b)
    h.close()
