"""Clusters seen only through pinholes of what is drawn before them: footprints of every width and height, tested in one
pass of 64 pixels or several.  And triangles across several frustum planes, more of them at once than the general clipper
takes at a time.  Frames are the oracle's, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

P = np.array([[1, 0, 0, 0], [0, 1, 0, 0], [0, 0, 20 / 19.99, -.2 / 19.99], [0, 0, 1, 0]])      # looks along +z, 90 degrees


def grid(c0, c1, z, n):
    """n x n quads between two corners in the plane at depth z (coordinates at depth 1)."""
    x, y = (np.linspace(c0[k], c1[k], n + 1) * z for k in (0, 1))
    v = np.stack([np.tile(x, n + 1), np.repeat(y, n + 1), np.full((n + 1) ** 2, z)], 1)
    q = (np.arange(n)[:, None] * (n + 1) + np.arange(n)).reshape(-1, 1)
    return v, np.concatenate([q + [0, 1, n + 1], q + [1, n + 2, n + 1]])


def mesh(parts):
    at, V, T = 0, [], []
    for v, t in parts:
        V.append(v)
        T.append(t + at)
        at += len(v)
    return np.concatenate(V).astype(np.float32), np.concatenate(T).astype(np.uint32)


def check(v, t, M, H, W, **cfg):
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    ref = oracle.render_scene(v, t, M, H, W)
    with bps.Renderer(max_batch=len(M), height=H, width=W, **cfg) as r:
        h = r.load_scene(v, t)
        depth, _, tid = r.render(np.full(len(M), h, np.int32), M, want_tri_id=True)
        torch.cuda.synchronize()
        assert np.array_equal(tid.cpu().numpy().view(np.uint32), ref["tri_id"])
        assert np.array_equal(depth.cpu().numpy(), ref["depth"])
    return ref


@pytest.mark.parametrize("w,h", [(1, 1), (1, 32), (2, 31), (3, 17), (4, 16), (5, 9), (8, 8), (9, 8), (17, 5), (32, 2), (32, 3), (32, 32), (33, 4)])
@pytest.mark.parametrize("frame", [(64, 64), (128, 128), (56, 88)])
def test_footprints_behind_pinholes(w, h, frame):
    H, W = frame
    rng = np.random.default_rng(64 * w + h)
    parts = []
    for j in range(H):      # a wall of one quad per pixel, one in a hundred missing
        for i in range(W):
            if rng.random() > 0.01:
                parts.append(grid((2 * i / W - 1, 2 * j / H - 1), (2 * (i + 1) / W - 1, 2 * (j + 1) / H - 1), 1.0, 1))
    for k in range(120):    # patches of w x h pixels behind it
        i, j = rng.uniform(0, W - w), rng.uniform(0, H - h)
        parts.append(grid((2 * i / W - 1, 2 * j / H - 1), (2 * (i + w) / W - 1, 2 * (j + h) / H - 1), 2.0 + 0.1 * k, 6))
    v, t = mesh(parts)
    ref = check(v, t, np.repeat(P[None], 2, 0).astype(np.float32), H, W)
    assert (ref["depth"] > 1.5).any()
    check(v, t, P[None].astype(np.float32), H, W, threads=384)


@pytest.mark.parametrize("n", [1, 3, 4, 7, 64, 65, 200])
def test_triangles_across_several_planes(n):
    rng = np.random.default_rng(n)
    far = rng.normal(size=(n, 3, 3)) * 30 + [0, 0, 8]
    v, t = mesh([(far.reshape(-1, 3), np.arange(3 * n).reshape(-1, 3))])
    a = rng.uniform(0, 2 * np.pi, 6)
    M = np.stack([P @ np.array([[np.cos(x), 0, np.sin(x), 0], [0, 1, 0, 0], [-np.sin(x), 0, np.cos(x), 0], [0, 0, 0, 1]]) for x in a]).astype(np.float32)
    for H, W in ((64, 64), (128, 128), (24, 72)):
        check(v, t, M, H, W)
