"""Streamed CSR rows (a group of 64 or 32 rows through LDS at a time): products
with row lengths from one to beyond a group's capacity, ragged ends, and groups
whose entries do not fit, entry by entry against a CSR product."""
import numpy as np
import pytest
import scipy.sparse as sp

from tests.gpu_helpers import dev_vec

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1403_1649_amd")

N = 65537   # the smallest size that is streamed: one row in the last group


def _rows(kind, n):
    rng = np.random.default_rng(5)
    if kind == "one":
        return np.ones(n, dtype=int)
    if kind == "seven":
        return np.full(n, 7)
    if kind == "thirteen":
        return rng.integers(1, 26, n)
    if kind == "burst":        # groups of 64 full rows of 40 among short ones
        c = np.full(n, 3)
        c[640:704] = 40
        c[-64:] = 40
        return c
    c = rng.integers(1, 6, n)  # "long": single rows of 1500 and 513 entries
    c[[7, n // 2, n - 1]] = 1500, 513, 1500
    return c


@pytest.mark.parametrize("extra", [0, 191])
@pytest.mark.parametrize("kind", ["one", "seven", "thirteen", "burst", "long"])
def test_streamed_product(kind, extra):
    n = N + extra
    cnt = _rows(kind, n)
    rp = np.zeros(n + 1, np.int32)
    np.cumsum(cnt, out=rp[1:])
    rng = np.random.default_rng(1)
    start = rng.integers(0, n - cnt)
    row = np.repeat(np.arange(n), cnt)
    col = (start[row] + (np.arange(rp[-1]) - rp[row])).astype(np.int32)
    val = rng.standard_normal(rp[-1])
    S = sp.csr_matrix((val, col, rp), shape=(n, n))
    x = rng.standard_normal(n)
    print(f"streamed {kind} n={n} nnz={rp[-1]}", flush=True)
    assert rp[-1] <= 15 * n
    y = amg.spmv(torch.from_numpy(rp).cuda(), torch.from_numpy(col).cuda(), dev_vec(val), dev_vec(x))
    # both sides sum at most max(cnt) products: each within that many roundings
    assert np.all(np.abs(y.cpu().numpy() - S @ x) <= 2.5e-16 * cnt.max() * (abs(S) @ np.abs(x)))
