"""bps_render_static, the entry point that allocates nothing (its launch plan lives in a static
__device__ array of the library), must fill the same frames as bps_render: checked through the
C ABI on two calls in a row, the second with a smaller batch (the array keeps the first call's
contents), then on a 128x128 renderer (four work-groups per frame) that reuses the same array."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _both(bps, torch, r, ids, vp):
    B = len(ids)
    d0 = torch.full((B, r.H, r.W), -1.0, dtype=torch.float32, device="cuda")
    i0 = torch.full((B, r.H, r.W), -2, dtype=torch.int32, device="cuda")
    d1, i1 = d0.clone(), i0.clone()
    bps.bps_render(r.handle, ids, vp, d0, out_tri_id=i0)
    bps.bps_render_static(r.handle, ids, vp, d1, out_tri_id=i1)
    torch.cuda.synchronize()
    return d0.cpu().numpy(), i0.cpu().numpy(), d1.cpu().numpy(), i1.cpu().numpy()


def test_static_entry_point_matches_bps_render_on_two_calls_in_a_row():
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    w = synth.build_config(2, B=700)          # more work-groups than two per compute unit: the planned path
    small = synth.build_config(1)             # 16 environments: the unplanned path, after the large call
    with bps.Renderer(max_batch=w.B, height=w.H, width=w.W) as r:
        h = r.load_scene(w.scenes[0].vertices, w.scenes[0].indices)
        h2 = r.load_scene(small.scenes[0].vertices, small.scenes[0].indices)
        vp = torch.from_numpy(w.view_proj).cuda()
        ids = np.full(w.B, h, np.int32)
        d0, i0, d1, i1 = _both(bps, torch, r, ids, vp)
        assert np.array_equal(i0, i1) and np.array_equal(d0.view(np.uint32), d1.view(np.uint32))
        # second call, smaller input, other scene
        vp2 = torch.from_numpy(small.view_proj).cuda()
        ids2 = np.full(small.B, h2, np.int32)
        e0, j0, e1, j1 = _both(bps, torch, r, ids2, vp2)
        assert np.array_equal(j0, j1) and np.array_equal(e0.view(np.uint32), e1.view(np.uint32))
        ref = oracle.render_batch(small.scenes, small.scene_ids, small.view_proj, small.H, small.W)
        assert np.array_equal(j1.view(np.uint32), ref["tri_id"])
        assert np.all(np.abs(e1 - ref["depth"]) <= 1e-5 * np.abs(ref["depth"]))
        # and the first input again: the array held the small plan in between
        d2 = torch.empty((w.B, w.H, w.W), dtype=torch.float32, device="cuda")
        bps.bps_render_static(r.handle, ids, vp, d2)
        torch.cuda.synchronize()
        assert np.array_equal(d2.cpu().numpy().view(np.uint32), d0.view(np.uint32))
    # a second renderer (128x128: four windows per frame) shares the device's array
    with bps.Renderer(max_batch=96, height=128, width=128) as r:
        h = r.load_scene(w.scenes[0].vertices, w.scenes[0].indices)
        vp = torch.from_numpy(w.view_proj[:96]).cuda()
        ids = np.full(96, h, np.int32)
        d0, i0, d1, i1 = _both(bps, torch, r, ids, vp)
        assert np.array_equal(i0, i1) and np.array_equal(d0.view(np.uint32), d1.view(np.uint32))


def test_static_entry_point_rejects_what_it_cannot_do():
    import torch
    import paper_2103_07013_amd as bps
    small = synth.build_config(1)
    vp_host = small.view_proj
    vp = torch.from_numpy(vp_host).cuda()
    depth = torch.empty((small.B, 64, 64), dtype=torch.float32, device="cuda")
    lib = bps.load_library()
    with bps.Renderer(max_batch=16, height=64, width=64) as r:
        h = r.load_scene(small.scenes[0].vertices, small.scenes[0].indices)
        ids = np.full(small.B, h, np.int32)
        # host matrices are refused (nothing may be staged), with an error text
        st = lib.bps_render_static(r.handle, ids.ctypes.data, vp_host.ctypes.data, small.B, depth.data_ptr(), None, None)
        assert st == -1 and "device memory" in bps.bps_last_error(r.handle)
        bad = ids.copy()
        bad[3] = 77
        with pytest.raises(bps.BpsError) as e:
            bps.bps_render_static(r.handle, bad, vp, depth)
        assert e.value.status == -2
    with bps.Renderer(max_batch=16, height=64, width=64, mode=bps.MODE_RGBD) as r:
        h = r.load_scene(small.scenes[0].vertices, small.scenes[0].indices, small.scenes[0].colors)
        with pytest.raises(bps.BpsError) as e:
            bps.bps_render_static(r.handle, np.full(16, h, np.int32), vp, depth)
        assert e.value.status == -5
    # sizes beyond the static array: 128x128 frames need four work-groups each
    with bps.Renderer(max_batch=4100, height=128, width=128) as r:
        h = r.load_scene(small.scenes[0].vertices, small.scenes[0].indices)
        big_vp = torch.zeros((4100, 4, 4), dtype=torch.float32, device="cuda")
        big_d = torch.empty((4100, 128, 128), dtype=torch.float32, device="cuda")
        with pytest.raises(bps.BpsError) as e:
            bps.bps_render_static(r.handle, np.full(4100, h, np.int32), big_vp, big_d)
        assert e.value.status == -1 and "static scratch" in str(e.value)


@pytest.mark.parametrize("first", [0, 1])
def test_static_entry_point_of_renderers_one_after_the_other(first):
    """A renderer that is made when another one is gone, for a scene whose frames are cut differently: its first
    plan is its own (tests/test_launch_plans.py checks the items themselves)."""
    import torch
    import paper_2103_07013_amd as bps
    B = 300
    scenes = [synth.make_multiroom_scene(T, seed=40 + T % 7) for T in (10_000, 100_000)]
    for s in (scenes[first], scenes[1 - first], scenes[first]):
        vp = torch.from_numpy(synth.make_cameras(s, B, seed=8)[0]).cuda()
        with bps.Renderer(max_batch=B) as r:
            ids = np.full(B, r.load_scene(s.vertices, s.indices), np.int32)
            d1 = torch.full((B, 64, 64), -1.0, dtype=torch.float32, device="cuda")
            i1 = torch.full((B, 64, 64), -2, dtype=torch.int32, device="cuda")
            bps.bps_render_static(r.handle, ids, vp, d1, out_tri_id=i1)
            torch.cuda.synchronize()
            d0, i0 = torch.empty_like(d1), torch.empty_like(i1)
            bps.bps_render(r.handle, ids, vp, d0, out_tri_id=i0)
            torch.cuda.synchronize()
            assert torch.equal(i0, i1) and torch.equal(d0, d1)


@pytest.mark.parametrize("B", [5, 300, 700])
def test_static_entry_point_captured_into_a_graph(B):
    """One batch cut into small windows, one into halves, one with planning kernels.  Every replay reads the matrices
    as they are then; calls made at once, with the captured plan and with another one, and synchronizations lie between."""
    import torch
    import paper_2103_07013_amd as bps
    s = synth.make_multiroom_scene(100_000, seed=43)
    poses = [torch.from_numpy(synth.make_cameras(s, B, seed=50 + k)[0]).cuda() for k in range(4)]
    with bps.Renderer(max_batch=B) as r:
        ids = np.full(B, r.load_scene(s.vertices, s.indices), np.int32)
        ref = []
        for p in poses:
            d, _, t = r.render(ids, p, want_tri_id=True)
            ref.append((d.clone(), t.clone()))
        torch.cuda.synchronize()
        vp = poses[0].clone()
        d1 = torch.empty((B, 64, 64), dtype=torch.float32, device="cuda")
        i1 = torch.empty((B, 64, 64), dtype=torch.int32, device="cuda")
        d2, i2 = torch.empty_like(d1), torch.empty_like(i1)

        def at_once(n, p):
            bps.bps_render_static(r.handle, ids[:n], poses[p][:n], d2[:n], out_tri_id=i2[:n])
            torch.cuda.synchronize()
            assert torch.equal(d2[:n], ref[p][0][:n]) and torch.equal(i2[:n], ref[p][1][:n])

        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            bps.bps_render_static(r.handle, ids, vp, d1, out_tri_id=i1)
        at_once(B, 1)
        for k, p in enumerate((0, 1, 2, 3, 2)):
            vp.copy_(poses[p])
            d1.fill_(-1.0)
            i1.fill_(-2)
            graph.replay()
            if k % 2:
                at_once(B, 3)                 # the plan of the graph
                at_once(max(1, B // 3), 2)    # and another one
            torch.cuda.synchronize()
            assert torch.equal(d1, ref[p][0]) and torch.equal(i1, ref[p][1]), f"replay {k}"
