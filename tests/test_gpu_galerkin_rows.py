"""The Galerkin product's rows by size: term counts on either side of what the
passes hold (128, 256 and 512 terms in the first, chosen by the average row,
1,024 in the wide one, and the extraction beyond), aggregates of more members
than a row's lanes, and fine rows longer than eight entries.  Against the
oracle's product, whose entries sum the same terms: 1e-14 of the row's absolute
terms times their number covers any order of summation."""
import numpy as np
import pytest
import scipy.sparse as sp

from oracle import amg_oracle as O
from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1403_1649_amd")


def _matrix(n, row_lens, seed):
    """Symmetric pattern with a diagonal and about row_lens[i] entries in row i."""
    rng = np.random.default_rng(seed)
    rows = np.repeat(np.arange(n), np.maximum(row_lens - 1, 0) // 2)
    S = sp.coo_matrix((rng.uniform(-1, 1, rows.size), (rows, rng.integers(0, n, rows.size))), shape=(n, n)).tocsr()
    S = (S + S.T + sp.identity(n) * 50).tocsr()
    S.sort_indices()
    return S


@pytest.mark.parametrize("per_row,members", [(5, 25), (5, 26), (9, 14), (9, 28), (17, 15), (17, 30), (17, 60), (33, 31),
                                             (65, 70), (3, 1)])
def test_rows_near_the_passes_limits(per_row, members):
    """Aggregates of members +- 1 rows: term counts around per_row * members."""
    rng = np.random.default_rng(per_row * 100 + members)
    sizes = np.concatenate([np.full(12, members - 1), np.full(12, members), np.full(12, members + 1), [1, 2, 3]])
    sizes = sizes[sizes > 0]
    n, nc = int(sizes.sum()), len(sizes)
    S = _matrix(n, np.full(n, per_row), members)
    A = P.CSR(S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)
    agg = rng.permutation(np.repeat(np.arange(nc), sizes)).astype(np.int32)
    pval = rng.uniform(0.5, 1.5, n)
    terms = np.bincount(agg, weights=np.diff(S.indptr), minlength=nc)
    print(f"galerkin rows: {per_row} x {members}, terms {terms.min():.0f} to {terms.max():.0f}", flush=True)
    rp, ci, v = to_dev(A)
    got_rp, got_ci, got_v = amg.galerkin(rp, ci, v, torch.from_numpy(agg).cuda(), dev_vec(pval), nc)
    want = O.galerkin(S, agg.astype(np.int64), pval, nc)
    size = O.galerkin(abs(S), agg.astype(np.int64), pval, nc)
    assert np.array_equal(got_rp, want.indptr) and np.array_equal(got_ci, want.indices)
    assert np.all(np.abs(got_v - want.data) <= 2.3e-16 * (terms.max() + 2) * size.data)
