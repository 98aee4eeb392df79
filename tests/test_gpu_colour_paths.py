"""GPU parity of the colour pass's paths: whole triangles, one clip plane, several, and what only the general path takes."""
import numpy as np
import pytest

from test_gpu_triangle_paths import _soup

pytestmark = pytest.mark.gpu


def _scene():
    """Random triangles and slivers across every plane; 24 wedges from outside a frame corner, more different
    triangles that cross two planes than one pass of the clipper takes; triangles from edge to edge."""
    v, _ = _soup(5, 700, 0.3, 1.2)
    ang = np.deg2rad(np.linspace(12, 78, 25))
    z = np.linspace(0.05, 0.06, 24)
    p0 = np.array([-1.05, -1.05])
    tip = p0 + 0.5 * np.stack([np.cos(ang), np.sin(ang)], 1)
    wedges = np.stack([np.concatenate([np.broadcast_to(p0, (24, 2)), z[:, None]], 1), np.concatenate([tip[:-1], z[:, None]], 1),
                       np.concatenate([tip[1:], z[:, None]], 1)], 1)
    wide = np.array([[[-1, -1, 0.95], [1, -1, 0.95], [1, 1, 0.95]], [[-1, -1, 0.95], [1, 1, 0.95], [-1, 1, 0.95]],
                     [[-5, -4, 0.97], [6, -3, 0.99], [0, 7, 0.9]]])
    v = np.concatenate([v.reshape(-1, 3, 3), wedges, wide]).reshape(-1, 3).astype(np.float32)
    return v, np.arange(v.shape[0], dtype=np.uint32).reshape(-1, 3)


def _matrices(B):
    Ms = np.zeros((B, 4, 4), np.float32)
    for k in range(B):
        c = np.float32(2.0) ** [0, 0, 0, 0, -58, 58, -62, 62, 0, 0, 0][k]
        Ms[k, 0, 0] = c * [1, -1, 1, 1, 1, 1, 1, 1, 1, 0.6, 3][k]
        Ms[k, 1, 1] = c * [1, 1, -1, 1, 1, 1, 1, 1, 1, 0.6, 3][k]
        Ms[k, 2, 2], Ms[k, 2, 3] = [(0.4 * c, 0.5 * c), (1.7 * c, -0.6 * c)][k % 2]      # every second one cut by near and far
        Ms[k, 3] = [(0, 0, 0, c), (0.3 * c, 0.1 * c, 0.2 * c, 1.2 * c)][k // 2 % 2]
    return Ms


@pytest.mark.parametrize("H,W", [(64, 64), (72, 104), (8, 8), (128, 128)])
def test_colours_through_every_path(H, W):
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    v, idx = _scene()
    rng = np.random.default_rng(8)
    B = 11
    Ms = _matrices(B)
    colors = rng.integers(0, 256, (len(v), 3)).astype(np.uint8)
    colors[::5] = 0
    colors[1::5] = 255
    ref = oracle.render_scene(v, idx, Ms, H, W, colors=colors)
    with bps.Renderer(max_batch=B, height=H, width=W, mode=bps.MODE_RGBD) as r:
        h = r.load_scene(v, idx, colors)
        depth = torch.empty((B, H, W), device="cuda")
        room = torch.full((B * H * W * 3 + 8,), 77, dtype=torch.uint8, device="cuda")
        for shift in (0, 1, 4):                       # 1: not on a word's boundary
            rgb = room[shift:shift + B * H * W * 3].view(B, H, W, 3)
            r.render(np.full(B, h, np.int32), Ms, out_depth=depth, out_rgb=rgb)
            torch.cuda.synchronize()
            assert np.array_equal(depth.cpu().numpy(), ref["depth"])
            bad = (rgb.cpu().numpy() != ref["rgb"]).any(-1)
            assert not bad.any(), f"shift {shift}: {int(bad.sum())} pixels differ, first at {np.argwhere(bad)[:4].tolist()}"
            assert (room[shift + B * H * W * 3:] == 77).all()
            room.fill_(77)


@pytest.mark.parametrize("bilinear", [False, True])
@pytest.mark.parametrize("scale,th,tw", [(1.0, 32, 64), (40.0, 256, 1), (1e-25, 16, 16), (1e24, 16, 16), (900.0, 512, 512)])
def test_texture_coordinates_of_every_size(scale, th, tw, bilinear):
    """Coordinates whose quotients leave the short division's range, exact zeros, levels far below the smaller side."""
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    v, idx = _scene()
    rng = np.random.default_rng(9)
    B = 11
    Ms = _matrices(B)
    uvs = (rng.uniform(-1, 1, (len(v), 2)) * scale).astype(np.float32)
    uvs[::7] = 0.0
    uvs[1::7, 0] = 0.0
    uvs[600:900] = 0.0
    tex = rng.integers(0, 256, (th, tw, 3)).astype(np.uint8)
    ref = oracle.render_scene(v, idx, Ms, 64, 64, uvs=uvs, texture=tex, bilinear=bilinear)
    with bps.Renderer(max_batch=B, mode=bps.MODE_RGBD, flags=bps.FLAG_BILINEAR if bilinear else 0) as r:
        h = r.load_scene_textured(v, idx, uvs, tex)
        _, rgb, tid = r.render(np.full(B, h, np.int32), Ms, want_tri_id=True)
        torch.cuda.synchronize()
    assert np.array_equal(tid.cpu().numpy().view(np.uint32), ref["tri_id"])
    bad = (rgb.cpu().numpy() != ref["rgb"]).any(-1)
    assert not bad.any(), f"{int(bad.sum())} pixels differ, first at {np.argwhere(bad)[:4].tolist()}"
