"""Streamed CSR rows whose groups exceed what a wave holds at a time: groups one
entry either side of the limit, rows beyond the limit, empty rows, uneven and
power-law lengths, in groups of 64 and of 32 rows."""
import numpy as np
import pytest
import scipy.sparse as sp

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1403_1649_amd")

N = 65536 + 77   # the smallest streamed size, a ragged last group


def _lengths(kind, mean, rng):
    """Row lengths of about `mean` on average (up to 7: groups of 64 rows, from 8
    of 32; beyond 30 lanes)."""
    l = np.full(N, mean)
    if kind == "uneven":
        l = rng.integers(0, 2 * mean + 1, N)
        l[5] += max(0, N - l.sum())
    elif kind == "limit":       # groups of 64 rows with 511, 512 and 513 entries, and of 32 rows as well
        l[:] = max(mean - 1, 1)
        for g, total in enumerate((511, 512, 513, 512, 1025)):
            l[64 * g:64 * g + 32] = 0
            l[64 * g:64 * g + 31] = total // 31
            l[64 * g + 31] = total - 31 * (total // 31)
            l[64 * g + 32:64 * g + 64] = 0
        l[-1] += 64 * 5
    elif kind == "long":        # single rows of 64, 65, 512, 513 and 3000 entries among short ones
        l[:] = max(mean - 1, 1)
        at = rng.choice(N, 200, replace=False)
        l[at] = rng.choice([64, 65, 512, 513, 3000], 200)
        l[[0, 63, 64, N - 1]] = [600, 65, 700, 900]
    elif kind == "power":
        l = np.minimum(4000, (rng.uniform(size=N) ** -0.8).astype(int))
        l = np.maximum(l, max(mean // 2, 1))
    return l


@pytest.mark.parametrize("mean", [1, 2, 3, 4, 5, 7, 9, 13, 16, 18, 29, 34])
@pytest.mark.parametrize("kind", ["even", "uneven", "limit", "long", "power"])
def test_groups_beyond_the_limit(kind, mean):
    rng = np.random.default_rng(mean)
    l = _lengths(kind, mean, rng)
    rp = np.concatenate([[0], np.cumsum(l)]).astype(np.int32)
    nnz = int(rp[-1])
    assert nnz >= N
    row = np.repeat(np.arange(N), l)
    ci = ((row + (np.arange(nnz) - rp[row]) * 7) % N).astype(np.int32)
    val = rng.standard_normal(nnz)
    x = rng.standard_normal(N)
    print(f"stream groups: {kind} {mean} nnz/n={nnz / N:.2f}", flush=True)
    dev = [torch.from_numpy(a).cuda() for a in (rp, ci, val, x)]
    y = amg.spmv(*dev).cpu().numpy()
    S = sp.csr_matrix((val, ci, rp), shape=(N, N))
    mag = sp.csr_matrix((np.abs(val), ci, rp), shape=(N, N)) @ np.abs(x)
    # both sides sum a row's products, each within (count - 1) u of the exact row sum
    assert np.all(np.abs(y - S @ x) <= 2.3e-16 * np.maximum(l, 1) * mag)
    assert np.array_equal(y, amg.spmv(*dev).cpu().numpy())
