"""Triangles that cross three and more planes, of which the general clipper takes eight at a time, and four of those whose
polygons turn out to have more than eight corners: as many of them as make a pass full, short by one and over by one.  Frames are the oracle's, bit for bit."""
import numpy as np
import pytest

from test_gpu_triangle_paths import NOHIT, _check

pytestmark = pytest.mark.gpu


def across(n, seed, corners=0.3):
    """n triangles around the middle of the view volume that reach far beyond its sides (its corners cut by a third of
    them, which leaves polygons of up to nine corners), and matrices that see them whole, from within and in perspective."""
    rng = np.random.default_rng(seed)
    a = rng.uniform(0, 2 * np.pi, (n, 1)) + np.array([0, 2.1, 4.2]) + rng.uniform(-.5, .5, (n, 3))
    r = np.where(rng.random((n, 1)) < corners, rng.uniform(1.7, 2.6, (n, 3)), rng.uniform(3, 40, (n, 3)))
    v = np.stack([r * np.cos(a), r * np.sin(a), .5 + rng.uniform(-1.5, 1.5, (n, 3)) * (rng.random((n, 1)) < .7)], 2)
    M = np.zeros((4, 4, 4), np.float32)
    M[:, 0, 0], M[:, 1, 1], M[:, 2, 2], M[:, 3, 3] = 1, 1, 1, 1
    M[1, 3, 2], M[1, 2, 3] = 1.0, -0.25
    M[2, 0, 3], M[2, 1, 3] = .3, -.4
    M[3, 3, 0], M[3, 3, 1] = .02, -.015
    return v.reshape(-1, 3).astype(np.float32), np.arange(3 * n, dtype=np.uint32).reshape(n, 3), M


@pytest.mark.parametrize("n", [1, 3, 4, 5, 7, 8, 9, 63, 64, 65, 300])
@pytest.mark.parametrize("H,W,copies", [(64, 64, 1), (64, 64, 150), (128, 128, 1), (72, 104, 9)])
def test_numbers_of_triangles(n, H, W, copies):
    v, t, M = across(n, n)
    ids = _check(v, t, np.tile(M, (copies, 1, 1)), H, W)
    assert (ids != NOHIT).mean() > .2


def test_triangles_are_fetched_once():
    """What a run of the clipper holds (64 triangles when it starts before the list of clusters ends) does not depend on
    how many of them cross several planes."""
    import torch
    import paper_2103_07013_amd as bps
    v, t, M = across(4000, 7, corners=0)
    groups = []
    with bps.Renderer(max_batch=4, height=64, width=64, splits=1, flags=bps.FLAG_NO_OCCLUSION_CULL) as r:
        h = r.load_scene(v, t)
        for mode in (1, 4):
            bps.bps_set_diagnostics(r.handle, mode)
            r.render(np.full(4, h, np.int32), M)
            torch.cuda.synchronize()
            groups.append(bps.bps_read_diagnostics(r.handle).reshape(-1, 16))
    straddling, runs = int(groups[0][:, 3].sum()), int(groups[1][:, 9].sum())
    assert straddling > 8000
    assert runs <= straddling / 16, (straddling, runs)      # (half the wavefronts may leave a few each at the end)
