"""Small batches are cut into windows of the frame, down to 8x8 pixels: parity at every size a window can have."""
import numpy as np
import pytest

import synth
from test_gpu_triangle_paths import _soup

pytestmark = pytest.mark.gpu


def _scene_and_cameras(kind, B, aspect):
    if kind == "soup":              # every clip plane and window border crossed, no connectivity
        v, idx = _soup(7, 900, 0.4, 1.3)
        rng = np.random.default_rng(3)
        M = np.zeros((B, 4, 4), np.float32)
        M[:, 0, 0] = M[:, 1, 1] = rng.uniform(0.7, 1.6, B)
        M[:, 2, 2], M[:, 2, 3] = 0.4, 0.5
        M[:, 3, 3], M[:, 3, 2] = 1.2, 0.4
        return v, idx, M
    s = synth.make_multiroom_scene(60_000, seed=21, jitter=0.3)
    return s.vertices, s.indices, synth.make_cameras(s, B, seed=5, aspect=aspect)[0]


# batch sizes on both sides of where a window is halved once more, frames whose halves are uneven, that are one
# window wide or high, or smaller than a window
@pytest.mark.parametrize("kind", ["soup", "rooms"])
@pytest.mark.parametrize("H,W", [(64, 64), (128, 128), (72, 104), (8, 128), (8, 8), (40, 24), (120, 56)])
def test_windows_match_oracle(kind, H, W):
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    Bs = (1, 2, 9, 17, 70)
    v, idx, M = _scene_and_cameras(kind, max(Bs), W / H)
    ref = oracle.render_scene(v, idx, M, H, W)
    groups = []
    with bps.Renderer(max_batch=max(Bs), height=H, width=W) as r:
        h = r.load_scene(v, idx)
        vp = torch.from_numpy(M).cuda()
        for B in Bs:
            ids = np.full(B, h, np.int32)
            depth, _, tid = r.render(ids, vp[:B], want_tri_id=True)
            groups.append(bps.bps_query(r.handle, h, 5))
            d2, t2 = torch.empty_like(depth), torch.empty_like(tid)
            bps.bps_render_static(r.handle, ids, vp[:B], d2, t2)
            torch.cuda.synchronize()
            t = tid.cpu().numpy().view(np.uint32)
            bad = t != ref["tri_id"][:B]
            assert not bad.any(), f"B={B}: {int(bad.sum())} ids differ, first at {np.argwhere(bad)[:4].tolist()}"
            assert np.array_equal(depth.cpu().numpy(), ref["depth"][:B])
            assert torch.equal(depth, d2) and torch.equal(tid, t2)
    whole = ((H + 63) // 64) * ((W + 63) // 64)
    # one frame is cut as finely as 64 windows allow (the numbers themselves: test_launch_plans.py)
    eighths = (H // 8) * (W // 8)
    assert groups[0] == eighths if eighths <= 64 and max(H, W) <= 64 else whole < groups[0] <= 64
    assert all(g % B == 0 and B * whole <= g <= 64 * B for g, B in zip(groups, Bs))


def test_windows_colour_and_supersampling():
    """The colour pass and the box filter after a frame drawn as small windows: equal to large batches' frames."""
    import torch
    import paper_2103_07013_amd as bps
    s = synth.make_multiroom_scene(30_000, seed=22)
    cams = torch.from_numpy(synth.make_cameras(s, 600, seed=6)[0]).cuda()
    for ss in (1, 2):
        with bps.Renderer(max_batch=600, mode=bps.MODE_RGBD, supersample=ss) as r:
            h = r.load_scene(s.vertices, s.indices, s.colors)
            d, c, _ = r.render(np.full(600, h, np.int32), cams)
            assert bps.bps_query(r.handle, h, 5) == 600 * (4 if ss == 2 else 1)
            d3, c3, _ = r.render(np.full(3, h, np.int32), cams[:3])
            assert bps.bps_query(r.handle, h, 5) == 3 * 64
            torch.cuda.synchronize()
            assert torch.equal(d[:3], d3) and torch.equal(c[:3], c3)


@pytest.mark.parametrize("threads,diagnostics", [(256, 0), (384, 0), (1024, 0), (512, 1), (256, 2), (1024, 4)])
@pytest.mark.parametrize("H,W", [(64, 64), (72, 104)])
def test_windows_of_other_group_sizes_and_with_diagnostics(threads, diagnostics, H, W):
    """The instances with a layout chosen at run time take survivors by way of their order: batches cut into small
    windows and whole ones, lists with and without an order (more than 64 survivors), several rounds."""
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    v, idx, M = _scene_and_cameras("rooms", 60, W / H)
    ref = oracle.render_scene(v, idx, M, H, W)
    with bps.Renderer(max_batch=1400, height=H, width=W, threads=threads) as r:
        h = r.load_scene(v, idx)
        bps.bps_set_diagnostics(r.handle, diagnostics)
        whole = ((H + 63) // 64) * ((W + 63) // 64)
        for B in (1, 9, 60, 1400):      # 8 x 60 windows of 72x104 fit 2.1 groups per compute unit
            d, _, t = r.render(np.full(B, h, np.int32), np.resize(M, (B, 4, 4)), want_tri_id=True)
            groups = bps.bps_query(r.handle, h, 5)
            assert groups == B * whole if B == 1400 else groups > B * whole
            torch.cuda.synchronize()
            t, d = t.cpu().numpy().view(np.uint32), d.cpu().numpy()
            for at in range(0, B, 60):
                n = min(60, B - at)
                assert np.array_equal(t[at:at + n], ref["tri_id"][:n]), f"B={B}"
                assert np.array_equal(d[at:at + n], ref["depth"][:n]), f"B={B}"
