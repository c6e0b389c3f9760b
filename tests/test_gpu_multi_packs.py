"""Block solves by 16-byte packs of columns: column counts that fill a pack, leave
a remainder or fall back to single values (odd counts, a right-hand side that is
not 16-byte aligned), on a level that streams T with 16-bit columns and on small
ones.  Each column against its own single solve: the contract's residual, and x
to 1e-6 (what the stopping tolerance leaves where the counts differ)."""
import numpy as np
import pytest

from synthetic import problems as P
from tests.gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
amg = pytest.importorskip("paper_1403_1649_amd")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("cols", [1, 2, 3, 4, 6, 8, 33, 64])
def test_columns_match_single_solves(cols, precision):
    A = P.hetero3d(42, seed=4)   # 74,088 rows
    rng = np.random.default_rng(cols)
    B = rng.standard_normal((A.n, cols))
    print(f"packs: {cols} {precision}", flush=True)
    h = amg.setup(*to_dev(A), amg.Options(dim=3, precision=precision))
    S = A.to_scipy()
    room = torch.empty(A.n * cols + 1, dtype=torch.float64, device="cuda")
    for shift in (0, 1):   # the second starts 8 bytes past a 16-byte boundary
        b = room[shift:shift + A.n * cols].view(A.n, cols)
        b.copy_(torch.from_numpy(B))
        x = amg.solve_multi(h, b, 1e-8)[0].cpu().numpy()
        r = np.linalg.norm(B - S @ x, axis=0) / np.linalg.norm(B, axis=0)
        assert np.all(r <= 1.01e-8), r.max()
        for c in {0, cols // 2, cols - 1}:
            x1 = amg.solve(h, torch.from_numpy(B[:, c].copy()).cuda(), 1e-8)[0].cpu().numpy()
            assert np.linalg.norm(x[:, c] - x1) <= 1e-6 * np.linalg.norm(x1)
    h.close()
