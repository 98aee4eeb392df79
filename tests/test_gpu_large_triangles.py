"""Triangles that a whole wavefront draws, tile by tile: sizes around the tiles' edges, slivers, boxes that the window
cuts, and the two forms of the path (packed coordinates, and the general one for 1/w out of the short division's range)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _triangles(H, W, scale):
    """Pixel boxes from just above the medium class (8x8) up to the frame and past it, at unaligned places."""
    rng = np.random.default_rng(17)
    v = []
    for size in (8.2, 9.0, 12.0, 15.9, 16.1, 17.0, 24.0, 31.0, 33.0, 63.0, 64.5, 100.0, 140.0):
        for aspect in (1.0, 0.07, 14.0):
            for _ in range(4):
                at, ext = rng.uniform(-8.0, [W, H]), np.minimum([size * max(1.0, aspect), size / min(1.0, aspect)], 200.0) * [1.0, min(1.0, 1.0 / aspect)]
                p = at + ext * rng.choice([[[0, 0], [1, 0], [0, 1]], [[0, 0], [1, 1], [1, 0]], [[0, 0.3], [1, 0], [0.6, 1]]])
                w = rng.uniform(0.5, 3.0, 3) * scale
                v.append(np.stack([(2 * p[:, 0] / W - 1) * w, (2 * p[:, 1] / H - 1) * w, w], 1))
    v = np.concatenate(v).astype(np.float32)
    return v, np.arange(len(v), dtype=np.uint32).reshape(-1, 3)


@pytest.mark.parametrize("scale", [1.0, 2.0 ** 70])      # (2^70: depths beyond what div_in_range is used for)
@pytest.mark.parametrize("H,W", [(64, 64), (128, 128), (72, 104), (24, 120)])
def test_large_triangles_match_oracle(H, W, scale):
    import oracle
    import paper_2103_07013_amd as bps
    import torch
    v, idx = _triangles(H, W, scale)
    M = np.zeros((1, 4, 4), np.float32)      # clip = (x, y, w / 2, w)
    M[0, 0, 0] = M[0, 1, 1] = 1.0
    M[0, 2, 2], M[0, 3, 2] = 0.5, 1.0
    for B in (1, 600):                        # small windows, and whole ones
        with bps.Renderer(max_batch=B, height=H, width=W) as r:
            for first in range(0, len(idx), 26):      # few at a time, so that most of them stay visible
                part = idx[first:first + 26]
                ref = oracle.render_scene(v, part, M, H, W)
                h = r.load_scene(v, part)
                depth, _, tid = r.render(np.full(B, h, np.int32), np.repeat(M, B, 0), want_tri_id=True)
                torch.cuda.synchronize()
                assert (ref["tri_id"] != 0xFFFFFFFF).any()
                for b in (0, B - 1):
                    assert np.array_equal(tid[b].cpu().numpy().view(np.uint32), ref["tri_id"][0]), (B, first)
                    assert np.array_equal(depth[b].cpu().numpy(), ref["depth"][0]), (B, first)
                r.unload_scene(h)
