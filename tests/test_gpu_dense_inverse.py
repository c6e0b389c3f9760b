"""The coarsest operator's inverse, one launch per panel of 32 columns: sizes
around multiples of 32 (odd and even numbers of panels), and sizes whose
trailing tiles are too many for the fused pivot (a launch of its own for it
then).  A hierarchy of one level solves by that inverse alone: x against
numpy's, within n eps cond(A) of it for both."""
import numpy as np
import pytest
import scipy.sparse as sp

from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev

pytestmark = pytest.mark.gpu

amg = pytest.importorskip("paper_1403_1649_amd")


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 96, 97, 600, 1440, 1472, 1505])
def test_inverse_of_one_level(n):
    rng = np.random.default_rng(n)
    S = sp.random(n, n, density=min(1.0, 6.0 / n), random_state=rng, format="csr")
    S = S + S.T
    S = S + sp.diags(1.0 + np.asarray(abs(S).sum(axis=1)).ravel())   # dominant: eigenvalues in [1, 1 + 2 max sum]
    S = sp.csr_matrix(S)
    S.sort_indices()
    A = P.CSR(S.indptr.astype(np.int32), S.indices.astype(np.int32), S.data)
    b = rng.standard_normal(n)
    print(f"inverse n={n}", flush=True)
    h = amg.setup(*to_dev(A), amg.Options(dim=2, coarse_max=2048, dense_max=2048))
    assert h.num_levels() == 1
    x, it, rel = amg.solve(h, dev_vec(b), 1e-12)
    want = np.linalg.solve(S.toarray(), b)
    cond = np.linalg.cond(S.toarray())
    err = np.linalg.norm(x.cpu().numpy() - want) / np.linalg.norm(want)
    assert rel <= 1e-12 and it <= 2
    assert err <= 2 * n * np.finfo(float).eps * cond + 1e-12 * cond
    h.close()
