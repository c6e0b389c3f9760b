"""An error of the HIP runtime that is pending in the thread (as a launch that
failed leaves it) is reported by the solve, not cleared on the way: both outer
methods, and the solves after it are whole again."""
import numpy as np
import pytest

from synthetic import problems as P
from tests.gpu_helpers import dev_vec, to_dev

pytestmark = pytest.mark.gpu

amg = pytest.importorskip("paper_1403_1649_amd")


@pytest.mark.parametrize("flags", [0, amg.binding.FLAG_NO_GRAPH], ids=["graphs", "eager"])
@pytest.mark.parametrize("krylov", ["fcg", "fgmres"])
def test_pending_error_is_reported(krylov, flags):
    A = P.poisson2d(61, 47)
    b = P.rhs(A, P.exact_solution(A.n, 3))
    bd = dev_vec(b)
    h = amg.setup(*to_dev(A), amg.Options(dim=2, krylov=krylov, flags=flags))
    amg.solve(h, bd, 1e-8)
    x = dev_vec(np.zeros(A.n))
    hip = amg.lib()
    assert hip.hipSetDevice(1 << 20) != 0   # refused on the host; the error stays pending
    with pytest.raises(amg.AmgError):
        amg.solve(h, bd, 1e-8, x=x)
    hip.hipGetLastError()
    x, _, rel = amg.solve(h, bd, 1e-8, x=x)
    assert rel <= 1e-8
    assert np.linalg.norm(b - A.to_scipy() @ x.cpu().numpy()) <= 1.01e-8 * np.linalg.norm(b)
    h.close()
