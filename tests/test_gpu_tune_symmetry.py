"""The autotuner's decision for a shape depends on whether its matrix fits
symmetric diagonals: each kind has its own, whichever came first."""
import numpy as np
import pytest
import scipy.sparse as sp

from synthetic import problems as P
from tests.gpu_helpers import to_dev
from tests.test_gpu_post_operator import _csr
from tests.test_gpu_slices import _entrywise

pytestmark = pytest.mark.gpu

amg = pytest.importorskip("paper_1403_1649_amd")

N = 100   # 10^6 rows: symmetric diagonals take half the sliced ones' time


def _format(A, seed, **kw):
    h = amg.setup(*to_dev(A), amg.Options(dim=3, **kw))
    _entrywise(h, 0, seed)
    f = h.level_format(0)
    h.close()
    return f


def _skewed(S, last_only):
    """Values off their mirror images: above the diagonal everywhere, or one
    entry of the last row (which no sample of the rows can count on)."""
    v = np.array(S.val)
    row = np.repeat(np.arange(S.n), np.diff(S.row_ptr))
    at = np.flatnonzero(S.col > row)
    if last_only:
        at = at[-1:]
    v[at] *= 0.5
    return P.CSR(S.row_ptr, S.col, v)


@pytest.mark.parametrize("last_only, n", [(False, N), (True, N + 1)])
def test_each_kind_keeps_its_decision(last_only, n):
    S = P.poisson3d(n)
    A = _skewed(S, last_only)
    print(f"tune symmetry: n={n} last_only={last_only}", flush=True)
    first = _format(A, 91, krylov="fgmres")   # the shape's first setup is nonsymmetric
    assert first[0] != 5
    sym = _format(S, 92)
    assert sym[0] == 5
    assert _format(A, 93, krylov="fgmres") == first
    assert _format(S, 94) == sym


def test_no_diagonals_at_a_shape_tuned_to_them():
    """The same size, entries and row lengths in place, the inner nodes in
    random order: no diagonals, so the level is timed, not left untimed."""
    n = N + 2
    S = P.poisson3d(n)
    assert _format(S, 95)[0] == 5
    inner = np.flatnonzero(np.diff(S.row_ptr) == 7)
    p = np.arange(S.n)
    p[inner] = np.random.default_rng(3).permutation(inner)
    Q = sp.csr_matrix((np.ones(S.n), (np.arange(S.n), p)))
    A = _csr(Q @ S.to_scipy() @ Q.T)
    assert np.array_equal(A.row_ptr, S.row_ptr)
    sym_us = _format(S, 96)[2]
    first = _format(A, 97)
    assert first[0] in (0, 1, 2, 4) and first[2] != sym_us
    assert _format(A, 98) == first
    assert _format(S, 99)[0] == 5
