"""How a work-group's rounds begin: fewer blocks of 64 clusters than wavefronts, as many, one more, more than threads
take at a time (and one more than can be ordered); every group size; and the box tests on numbers far from one.  Frames are
the oracle's, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def patches(n, seed, scale=1.0):
    """n separate patches (a cluster each) of an 8x8 grid of vertices, in a box of 8 x 3 x 8 around the origin."""
    rng = np.random.default_rng(seed)
    g = np.stack(np.meshgrid(np.linspace(-.5, .5, 8), np.linspace(-.5, .5, 8)), -1).reshape(-1, 2)
    c, u, v = rng.uniform(-1, 1, (n, 1, 3)) * [4, 1.5, 4], rng.normal(size=(n, 1, 3)) * .2, rng.normal(size=(n, 1, 3)) * .2
    verts = (c + g[None, :, :1] * u + g[None, :, 1:] * v).reshape(-1, 3) * scale
    q = (np.arange(7)[:, None] * 8 + np.arange(7)).reshape(-1, 1)
    quads = np.concatenate([q + [0, 1, 8], q + [1, 9, 8]])
    tris = (64 * np.arange(n)[:, None, None] + quads).reshape(-1, 3)
    return verts.astype(np.float32), tris.astype(np.uint32)


def cameras(B, seed, scale=1.0):
    rng = np.random.default_rng(seed)
    P = np.array([[1, 0, 0, 0], [0, -1, 0, 0], [0, 0, -20 / 19.99, -.2 / 19.99], [0, 0, -1, 0]])
    out = np.empty((B, 4, 4), np.float32)
    for b in range(B):
        a, t = rng.uniform(0, 2 * np.pi), rng.uniform(-1, 1, 3) * [3, .5, 3]
        V = np.eye(4)
        V[:3, :3] = [[np.cos(a), 0, np.sin(a)], [0, 1, 0], [-np.sin(a), 0, np.cos(a)]]
        V[:3, 3] = -V[:3, :3] @ t
        out[b] = P @ V @ np.diag([1 / scale, 1 / scale, 1 / scale, 1])
    return out


def check(verts, tris, M, H, W, **cfg):
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    ref = oracle.render_scene(verts, tris, M, H, W)
    with bps.Renderer(max_batch=len(M), height=H, width=W, **cfg) as r:
        h = r.load_scene(verts, tris)
        depth, _, tid = r.render(np.full(len(M), h, np.int32), M, want_tri_id=True)
        torch.cuda.synchronize()
        assert np.array_equal(tid.cpu().numpy().view(np.uint32), ref["tri_id"])
        assert np.array_equal(depth.cpu().numpy(), ref["depth"])
    assert (ref["tri_id"] != 0xFFFFFFFF).any()


@pytest.mark.parametrize("clusters", [1, 64, 65, 8 * 64, 8 * 64 + 1, 16 * 64 + 1, 40 * 64])
@pytest.mark.parametrize("threads", [0, 256, 384, 512, 1024])
def test_numbers_of_blocks(clusters, threads):
    v, t = patches(clusters, clusters)
    for B, H, W in ((1, 64, 64), (3, 40, 88)):
        check(v, t, cameras(B, clusters + B), H, W, threads=threads)


@pytest.mark.parametrize("scale", [2.0 ** -40, 2.0 ** 60, 1e30])
def test_boxes_of_extreme_size(scale):
    v, t = patches(600, 7, scale)
    check(v, t, cameras(5, 3, scale), 64, 64)
    check(v, t, cameras(40, 4, scale), 48, 72)


def loose(n, seed):
    """n small triangles apart from each other (21 to a cluster) behind a wall that hides two thirds of them from +z."""
    rng = np.random.default_rng(seed)
    v = (rng.uniform(-1, 1, (n, 1, 3)) * [4, 1.5, 4] + rng.normal(size=(n, 3, 3)) * .04).reshape(-1, 3)
    g = np.stack(np.meshgrid(np.linspace(-4, 1, 8), np.linspace(-2, 2, 8)), -1).reshape(-1, 2)
    q = (np.arange(7)[:, None] * 8 + np.arange(7)).reshape(-1, 1)
    quads = np.concatenate([q + [0, 1, 8], q + [1, 9, 8]]) + len(v)
    wall = np.concatenate([g, np.full((64, 1), 4.5)], 1)
    return np.concatenate([v, wall]).astype(np.float32), np.concatenate([np.arange(3 * n).reshape(n, 3), quads]).astype(np.uint32)


@pytest.mark.parametrize("n,blocks,threads", [(345_000, 257, 256), (500_000, 373, 256), (500_000, 373, 384), (690_000, 514, 512),
                                              (690_000, 514, 256), (1_375_000, 1024, 512), (1_380_000, 1027, 256)])
def test_more_blocks_than_threads(n, blocks, threads):
    """One group on a whole scene (no windows, no shares), from where nearly all blocks are in view and from among them."""
    import paper_2103_07013_amd as bps
    v, t = loose(n, n)
    assert -(-len(bps.bps_pack_clusters(v, t)[0]) // 64) == blocks
    M = cameras(3, n)
    for b, z in enumerate((9, 12)):      # from outside, behind the wall
        P = np.array([[1, 0, 0, 0], [0, -1, 0, 0], [0, 0, -20 / 19.99, -.2 / 19.99], [0, 0, -1, 0]])
        V = np.eye(4)
        V[2, 3] = -z
        M[b] = P @ V
    check(v, t, M, 64, 64, threads=threads, splits=1)
