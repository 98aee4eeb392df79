"""Diagnostics count small and large triangles as the launch splits them that draws the request otherwise: one lane per
triangle up to 12 pixel centres in frames of 64x64 drawn whole, up to 20 in every other window."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def boxes(n, m, H, W, cuts):
    """Triangles whose boxes hold n x m pixel centres, apart from each other and from where the frame is cut."""
    tris = []
    for j in range(0, H - 7, 8):
        for i in range(0, W - 7, 8):
            if any(j < c < j + 8 for c in cuts[0]) or any(i < c < i + 8 for c in cuts[1]):
                continue
            p = [[i + 1.3, j + 1.3], [i + n + .7, j + 1.4], [i + 1.4, j + m + .7]]
            tris.append([[2 * x / W - 1, 2 * y / H - 1, .5] for x, y in p])
    v = np.array(tris, np.float32).reshape(-1, 3)
    return v, np.arange(len(v), dtype=np.uint32).reshape(-1, 3)


@pytest.mark.parametrize("H,W,B,cuts,limit", [(64, 64, 600, ((), ()), 12), (64, 64, 200, ((), ()), 20), (64, 64, 3, ((), ()), 20),
                                             (128, 128, 600, ((), ()), 20), (72, 104, 600, ((36,), (52,)), 20)])
@pytest.mark.parametrize("n,m", [(4, 3), (3, 4), (5, 3), (5, 4), (4, 5), (7, 3)])
def test_counts_of_small_and_large(H, W, B, cuts, limit, n, m):
    import torch
    import paper_2103_07013_amd as bps
    v, t = boxes(n, m, H, W, cuts)
    with bps.Renderer(max_batch=B, height=H, width=W) as r:
        ids = np.full(B, r.load_scene(v, t), np.int32)
        bps.bps_set_diagnostics(r.handle, 1)
        depth, _, _ = r.render(ids, np.broadcast_to(np.eye(4, dtype=np.float32), (B, 4, 4)).copy())
        torch.cuda.synchronize()
        words = bps.bps_read_diagnostics(r.handle, 1 << 18).reshape(-1, 16).sum(0)
    count = B * len(t)
    assert (int(words[6]), int(words[7])) == ((count, 0) if n * m <= limit else (0, count))
