"""Triangles whose box holds n x m pixel centres, on both sides of where one lane per triangle ends (12 centres in frames of
64x64, 20 in other windows) and at the edges of the 8x8 boxes after it.  Frames are the oracle's, bit for bit."""
import numpy as np
import pytest

from test_gpu_triangle_paths import NOHIT, _check

pytestmark = pytest.mark.gpu

SIZES = [(n, m) for n in range(1, 26) for m in range(1, 26) if 9 <= n * m <= 25 or (n, m) in ((8, 8), (9, 8), (8, 9))]


@pytest.mark.parametrize("H,W,B", [(64, 64, 1), (64, 64, 300), (128, 128, 2), (72, 104, 5)])
def test_numbers_of_centres(H, W, B):
    rng = np.random.default_rng(H + W + B)
    tris = []
    for n, m in SIZES * 6:
        i, j = rng.integers(0, W - n + 1), rng.integers(0, H - m + 1)
        lo, hi = np.array([i + rng.uniform(.05, .45), j + rng.uniform(.05, .45)]), np.array([i + n - rng.uniform(.05, .45), j + m - rng.uniform(.05, .45)])
        mid = rng.uniform(lo, hi)
        p = [[lo[0], lo[1]], [hi[0], mid[1]], [mid[0], hi[1]]] if rng.random() < .5 else [[lo[0], hi[1]], [hi[0], mid[1]], [mid[0], lo[1]]]
        tris.append([[2 * x / W - 1, 2 * y / H - 1, rng.uniform(.1, .9)] for x, y in p])
    v = np.array(tris).reshape(-1, 3).astype(np.float32)
    M = np.broadcast_to(np.eye(4, dtype=np.float32), (B, 4, 4)).copy()
    M[:, 3, 2] = np.linspace(0, .05, B)                     # (not all environments alike)
    M[:, 3, 2][0] = 0
    t = _check(v, np.arange(len(v), dtype=np.uint32).reshape(-1, 3), M, H, W)
    assert (t != NOHIT).mean() > .1
