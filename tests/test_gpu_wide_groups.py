"""Requests that put one group of sixteen wavefronts on a compute unit: parity where the rule for them begins and ends,
with one and with several rounds, with windows of every shape."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,T", [(64, 64, 120_000), (64, 64, 20_000), (128, 128, 400_000), (72, 104, 400_000), (8, 128, 60_000)])
def test_wide_groups_match_oracle(H, W, T):
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    Bs = (1, 2, 4, 5, 8, 17, 32, 33)
    s = synth.make_multiroom_scene(T, seed=41, jitter=0.3)
    M = synth.make_cameras(s, max(Bs), seed=6, aspect=W / H)[0]
    ref = oracle.render_scene(s.vertices, s.indices, M, H, W)
    wide_lds = []
    with bps.Renderer(max_batch=max(Bs), height=H, width=W) as r:
        h = r.load_scene(s.vertices, s.indices)
        many = 4 * bps.bps_query(r.handle, h, 0) >= H * W      # clusters rather than pixels
        vp = torch.from_numpy(M).cuda()
        for B in Bs:
            ids = np.full(B, h, np.int32)
            depth, _, tid = r.render(ids, vp[:B], want_tri_id=True)
            groups, lds = bps.bps_query(r.handle, h, 5), bps.bps_query(r.handle, h, 7)
            if groups <= cu:
                wide_lds.append(lds)
            assert groups % B == 0 and (groups <= cu or not many or 8 * B > cu)      # (eight windows a frame have to fit)
            d2, t2 = torch.empty_like(depth), torch.empty_like(tid)
            bps.bps_render_static(r.handle, ids, vp[:B], d2, t2)
            torch.cuda.synchronize()
            assert np.array_equal(tid.cpu().numpy().view(np.uint32), ref["tri_id"][:B]), f"B={B}"
            assert np.array_equal(depth.cpu().numpy(), ref["depth"][:B]), f"B={B}"
            assert torch.equal(depth, d2) and torch.equal(tid, t2), f"B={B}"
    assert len(set(wide_lds)) == 1 and wide_lds[0] > 82_000


@pytest.mark.parametrize("diagnostics", [1, 2, 4])
@pytest.mark.parametrize("H,W", [(64, 64), (72, 104)])
def test_wide_groups_with_diagnostics(H, W, diagnostics):
    """The records come from groups of the number and size that draw the request otherwise, and from the same frames."""
    import torch
    import oracle
    import paper_2103_07013_amd as bps
    s = synth.make_multiroom_scene(100_000, seed=41, jitter=0.3)
    M = synth.make_cameras(s, 17, seed=6, aspect=W / H)[0]
    ref = oracle.render_scene(s.vertices, s.indices, M, H, W)
    with bps.Renderer(max_batch=17, height=H, width=W) as r:
        h = r.load_scene(s.vertices, s.indices)
        for B in (1, 9, 17):
            ran = []
            for on in (0, diagnostics):
                bps.bps_set_diagnostics(r.handle, on)
                d, _, t = r.render(np.full(B, h, np.int32), M[:B], want_tri_id=True)
                torch.cuda.synchronize()
                ran.append((bps.bps_query(r.handle, h, 5), bps.bps_query(r.handle, h, 6)))
                assert np.array_equal(t.cpu().numpy().view(np.uint32), ref["tri_id"][:B]), (B, on)
                assert np.array_equal(d.cpu().numpy(), ref["depth"][:B]), (B, on)
            assert ran[0] == ran[1]
            words = bps.bps_read_diagnostics(r.handle).reshape(-1, 16)
            assert len(words) == ran[0][0] and words[:, 2].sum() > 0
            bps.bps_set_diagnostics(r.handle, 0)
