"""GPU parity of the raster kernel's triangle paths at the edges of what each of them takes."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
NOHIT = 0xFFFFFFFF


def _soup(seed, n, size, reach):
    """n random triangles: centres in [-reach, reach]^2, corners up to `size` away, plus long thin slivers from
    edge to edge of the frame."""
    rng = np.random.default_rng(seed)
    c = rng.uniform(-reach, reach, (n, 1, 3))
    t = c + rng.uniform(-size, size, (n, 3, 3))
    y = rng.uniform(-0.98, 0.98, (12, 1))
    x = np.where(np.arange(12)[:, None] % 2 == 0, [[-1.0, 1.0, 0.3]], [[-0.999, 0.998, -0.2]])
    h = rng.uniform(-0.02, 0.02, (12, 3))
    slivers = np.stack([x, np.clip(y + h, -1, 1), rng.uniform(0.1, 0.9, (12, 3))], 2)
    slivers = np.concatenate([slivers, slivers[:, :, [1, 0, 2]]])          # and from top to bottom
    v = np.concatenate([t, slivers]).reshape(-1, 3).astype(np.float32)
    return v, np.arange(v.shape[0], dtype=np.uint32).reshape(-1, 3)


def _check(v, idx, M, H, W, **kw):
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    ref = oracle.render_scene(v, idx, M, H, W)
    with bps.Renderer(max_batch=len(M), height=H, width=W, **kw) as r:
        h = r.load_scene(v, idx)
        depth, _, tid = r.render(np.full(len(M), h, np.int32), M, want_tri_id=True)
        torch.cuda.synchronize()
        d, t = depth.cpu().numpy(), tid.cpu().numpy().view(np.uint32)
    bad = t != ref["tri_id"]
    assert not bad.any(), f"{int(bad.sum())} ids differ, first at {np.argwhere(bad)[:4].tolist()}"
    assert np.array_equal(d, ref["depth"])
    return t


@pytest.mark.parametrize("H,W", [(64, 64), (128, 128), (72, 104), (8, 128)])
@pytest.mark.parametrize("size", [0.02, 0.15, 1.5])
def test_exponent_range_and_slivers(H, W, size):
    """Clip w far from 1: 2^-60 and 2^60 are the ends of the range in which depths are divided without the
    general division's scaling steps; frames stay equal to the oracle within it, at its ends, beyond it, and in
    batches whose matrices lie on both sides."""
    v, idx = _soup(int(1000 * size) + H, 600, size, 1.0)
    Ms = []
    for s in (0, -59, -60, -61, 59, 60, 61, -100, 100, -120, 120):
        c = np.float32(2.0) ** s
        M = np.zeros((4, 4), np.float32)
        M[0, 0] = M[1, 1] = c
        M[2, 2], M[2, 3] = 0.4 * c, 0.5 * c
        M[3] = [0.0, 0.0, 0.0, c]
        Ms.append(M.copy())
        M[3] = [0.25 * c, 0.0, 0.125 * c, 1.5 * c]      # perspective
        Ms.append(M)
    t = _check(v, idx, np.stack(Ms), H, W)
    assert (t != NOHIT).mean() > 0.02


@pytest.mark.parametrize("H,W,B", [(64, 64, 3), (128, 128, 2), (72, 104, 40), (64, 64, 600)])
@pytest.mark.parametrize("grid", [True, False])
def test_clipped_triangles(grid, H, W, B):
    """Triangles that cross one, two and more planes in every combination; on the grid many corners lie exactly on a
    plane, and pieces and whole triangles repeat (depth ties).  Both windings, few and many work-groups."""
    rng = np.random.default_rng(17)
    n = 1500
    if grid:
        v = np.stack([rng.choice([-1.5, -1.0, -0.5, 0.0, 0.25, 1.0, 2.0], (n, 3)), rng.choice([-2.0, -1.0, 0.0, 0.5, 1.0, 1.25], (n, 3)),
                      rng.choice([-0.25, 0.0, 0.25, 0.5, 1.0, 1.5], (n, 3))], 2)
    else:
        v = np.stack([rng.uniform(-1.6, 1.6, (n, 3)), rng.uniform(-1.6, 1.6, (n, 3)), rng.uniform(-0.4, 1.4, (n, 3))], 2)
        far = rng.random((n, 3)) < 0.1
        v[far] *= 10.0 ** rng.uniform(1, 6, (int(far.sum()), 1))
    v = v.reshape(-1, 3).astype(np.float32)
    idx = np.arange(3 * n, dtype=np.uint32).reshape(n, 3)
    M = np.zeros((B, 4, 4), np.float32)
    M[:, 0, 0], M[:, 1, 1], M[:, 2, 2], M[:, 3, 3] = 1, 1, 1, 1
    M[1::2, 3, 2], M[1::2, 2, 3] = 1.0, -0.25            # perspective: w = z + 1, near and far cut elsewhere
    M[2::3, 0, 0] = -1
    M[3:, 0, 3] = rng.uniform(-0.4, 0.4, max(B - 3, 0))
    t = _check(v, idx, M, H, W)
    assert (t != NOHIT).mean() > 0.3


def test_reciprocals_of_every_mantissa():
    """1/w in three instructions: one triangle of constant clip w per environment, w running through all 2^23 mantissas
    at one exponent and through every 251st of them at the others the short form takes.  A reciprocal off by its last
    bit changes some depth of the 8x8 frame for 99 % of them."""
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    v = np.array([[-0.9, -0.95, 0.2], [0.95, -0.7, 0.4], [-0.1, 0.9, 0.9]], np.float32)
    idx = np.array([[0, 1, 2]], np.uint32)
    one = 0x3F800000
    words = [np.arange(one, one + (1 << 23), dtype=np.uint32)]
    words += [np.arange(one + (e << 23), one + ((e + 1) << 23), 251, dtype=np.uint32) for e in (-60, -59, -31, -1, 1, 30, 58, 59)]
    words = np.concatenate(words)
    B = 1 << 16
    M = np.zeros((B, 4, 4), np.float32)
    with bps.Renderer(max_batch=B, height=8, width=8) as r:
        ids = np.full(B, r.load_scene(v, idx), np.int32)
        for at in range(0, len(words), B):
            w = np.resize(words[at:at + B], B).view(np.float32)
            M[:, 0, 0] = M[:, 1, 1] = M[:, 2, 2] = M[:, 3, 3] = w
            ref = oracle.render_scene(v, idx, M, 8, 8)
            depth, _, tid = r.render(ids, M, want_tri_id=True)
            torch.cuda.synchronize()
            assert np.array_equal(tid.cpu().numpy().view(np.uint32), ref["tri_id"])
            assert (ref["tri_id"] == 0).sum() == 26 * B
            bad = (depth.cpu().numpy() != ref["depth"]).any((1, 2))
            assert not bad.any(), f"{int(bad.sum())} of {B}, first w = {w[np.argmax(bad)]!r}"
