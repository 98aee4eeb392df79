"""The host side's launch plans, without a GPU: libbps.so runs on a stand-in for the HIP runtime (fake_hip.c), which
tells for every raster launch what the kernel would find in its work-item array."""
import os
import re
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PRELUDE = """
import ctypes, sys
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)      # found before the real runtime
fake.fake_log.restype = ctypes.c_char_p
import paper_2103_07013_amd as bps
import synth
lib = bps.load_library()
small = synth.make_multiroom_scene(10_000, seed=1)
large = synth.make_multiroom_scene(100_000, seed=2)
pool = np.zeros(1 << 16, np.float32)      # "device" matrices
fake.fake_device_range(ctypes.c_void_p(pool.ctypes.data), ctypes.c_size_t(pool.nbytes))
out = np.zeros(8, np.float32)             # never written: no kernel draws

def load(r, s):
    return bps.bps_load_scene(r, s.vertices, s.indices)

def static(r, h, B, offset=0):
    fake.fake_clear_log()
    ids = np.full(B, h, np.int32)
    assert lib.bps_render_static(r, ids.ctypes.data, pool[offset:].ctypes.data, B, out.ctypes.data, None, None) == 0, bps.bps_last_error(r)
    print(fake.fake_log().decode(), end="")
"""


CAPTURE = """
def capture(r, h, B):
    fake.fake_capture(1)
    static(r, h, B)
    fake.fake_capture(0)

def replay():
    fake.fake_clear_log()
    fake.fake_replay()
    print(fake.fake_log().decode(), end="")
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "fake_hip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-I/opt/rocm/include", os.path.join(ROOT, "tests", "fake_hip.c"), "-o", so],
                   check=True)
    return so


def _launches(fake, code):
    """The raster launches of the calls in `code`, as dicts."""
    p = subprocess.run([sys.executable, "-c", PRELUDE + code, fake], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr
    return [{k: int(v, 0) for k, v in re.findall(r"(\w+)=(\w+)", line)} for line in p.stdout.splitlines() if line.startswith("k_raster")]


@pytest.mark.parametrize("first,second", [("small", "large"), ("large", "small")])
def test_static_plan_of_a_renderer_that_is_gone(fake, first, second):
    """300 environments are drawn whole in the small scene and as halves in the large one.  The second renderer's
    handle may well be the address the first one had; its items must be its own all the same."""
    got = _launches(fake, f"""
for s in ({first}, {second}, {first}):
    r = bps.bps_create(max_batch=300)
    h = load(r, s)
    static(r, h, 300)
    static(r, h, 300)      # the same plan again
    bps.bps_destroy(r)
""")
    tiles = {"small": 1, "large": 2}
    assert [g["tiles"] for g in got] == [tiles[s] for s in (first, first, second, second, first, first)]
    assert all(g["wrong"] == 0 and g["envs"] == 300 and g["groups"] == 300 * g["tiles"] for g in got)


def test_static_plans_of_renderers_in_turn(fake):
    got = _launches(fake, """
a, b = bps.bps_create(max_batch=300), bps.bps_create(max_batch=300)
ha, hb = load(a, small), load(b, large)
for r, h, B in ((a, ha, 300), (b, hb, 300), (a, ha, 300), (b, hb, 17), (a, ha, 300), (b, hb, 17), (b, hb, 300)):
    static(r, h, B)
""")
    assert [g["envs"] for g in got] == [300, 300, 300, 17, 300, 17, 300]
    assert all(g["wrong"] == 0 and g["groups"] == g["envs"] * g["tiles"] for g in got)


def test_static_plans_of_captured_calls(fake):
    """A captured call writes nothing when it is made and everything on each replay."""
    got = _launches(fake, CAPTURE + """
r = bps.bps_create(max_batch=300)
hs, hl = load(r, small), load(r, large)
static(r, hs, 300)
capture(r, hl, 300)
static(r, hl, 300)      # the captured plan, which nothing has unpacked yet
replay()
static(r, hl, 17)       # another plan
replay()
static(r, hl, 17)       # the same again: the replay in between has left it alone
capture(r, hl, 17)      # a plan that the eager calls' array holds already
static(r, hs, 300)
replay()
static(r, hs, 300)
""")
    assert [g["envs"] for g in got] == [300, 300, 300, 17, 300, 17, 300, 17, 300]
    assert [g["tiles"] for g in got[:3]] == [1, 2, 2] and got[4]["tiles"] == 2 and got[6]["tiles"] == 1
    assert all(g["wrong"] == 0 and g["groups"] == g["envs"] * g["tiles"] for g in got)


@pytest.mark.parametrize("B", [17, 300])      # cut differently by the two entry points, and alike
def test_two_entry_points_in_turn_keep_their_plans(fake, B):
    got = _launches(fake, f"""
r = bps.bps_create(max_batch={B})
h = load(r, large)
ids = np.full({B}, h, np.int32)
for k in range(8):
    if k == 4:
        copied = fake.fake_copied()
    fake.fake_clear_log()
    assert lib.bps_render(r, ids.ctypes.data, pool.ctypes.data, {B}, out.ctypes.data, None, None, None) == 0
    print(fake.fake_log().decode(), end="")
    static(r, h, {B})
    if k >= 4:
        assert "k_unpack_items" not in fake.fake_log().decode()
assert fake.fake_copied() == copied
""")
    assert len(got) == 16 and all(g["wrong"] == 0 and g["envs"] == B for g in got)
    assert (got[0]["tiles"] == got[1]["tiles"]) == (B == 300)
    assert got[2:] == 7 * got[:2]


@pytest.mark.parametrize("B", [256, 257, 300, 2000])
def test_static_plan_stays_within_its_array_on_any_device(fake, B):
    """A device so large that the rule for small batches would like more groups than the array has items (16384)."""
    got = _launches(fake, f"""
fake.fake_compute_units(8192)
r = bps.bps_create(max_batch={B})
static(r, load(r, large), {B})
static(r, load(r, small), {B})
""")
    assert all(g["wrong"] == 0 and g["envs"] == B and g["groups"] == B * g["tiles"] and 16384 // 4 < g["groups"] <= 16384 for g in got)
    assert len(got) == 2 and all(1 < g["tiles"] <= 64 for g in got)


# the numbers of windows that halving along the longer side passes through, down to 8x8 pixels and up to 64 windows
HALVINGS = {(64, 64): [1, 2, 4, 8, 16, 32, 64], (128, 128): [4, 8, 16, 32, 64], (72, 104): [4, 8, 16, 32, 64],
            (8, 128): [2, 4, 8, 16], (8, 8): [1], (40, 24): [1, 2, 4, 8, 12, 15], (120, 56): [2, 4, 8, 16, 32, 60]}


@pytest.mark.parametrize("H,W", list(HALVINGS))
def test_windows_per_frame(fake, H, W):
    """Frames are halved as long as the groups fit 2 + clusters per window / 2048 per compute unit, at most 4.6."""
    import paper_2103_07013_amd as bps
    import synth
    scenes = [synth.make_multiroom_scene(10_000, seed=1), synth.make_multiroom_scene(100_000, seed=2)]
    clusters = [len(bps.bps_pack_clusters(s.vertices, s.indices)[0]) for s in scenes]
    Bs = (1, 2, 9, 17, 60, 70, 128, 256, 300, 319, 330, 587, 589, 2048)
    got = _launches(fake, f"""
r = bps.bps_create(max_batch=2048, height={H}, width={W})
hs = load(r, small), load(r, large)
for B in {Bs}:
    for h in hs:
        static(r, h, B)
""")
    for k, B in enumerate(Bs):
        for C, g in zip(clusters, got[2 * k:2 * k + 2]):
            want = HALVINGS[H, W][0]
            for finer in HALVINGS[H, W][1:]:
                if B * finer > 256 * min(2 + C / want / 2048, 4.6):
                    break
                want = finer
            assert g["tiles"] == want and g["wrong"] == 0 and g["groups"] == B * want, (B, C)


def test_windows_of_large_scenes(fake):
    """From 5300 clusters per window on the limit is 4.6 groups per compute unit: 588 frames are halved, 589 are not."""
    got = _launches(fake, """
r = bps.bps_create(max_batch=1024)
h = load(r, synth.make_multiroom_scene(600_000, seed=3))
assert bps.bps_query(r, h, 0) > 5400
for B in (588, 589, 1024):
    static(r, h, B)
""")
    assert [g["tiles"] for g in got] == [2, 1, 1] and all(g["wrong"] == 0 for g in got)


@pytest.mark.parametrize("threads", [0, 256, 384, 512, 1024])
def test_groups_have_the_size_that_was_asked_for(fake, threads):
    """Where none was, launches of one group per compute unit run 1024 threads and others 512."""
    got = _launches(fake, f"""
r = bps.bps_create(max_batch=300, threads={threads})
h = load(r, small)
for B in (1, 300):
    static(r, h, B)
    fake.fake_clear_log()
    ids = np.full(B, h, np.int32)
    assert lib.bps_render(r, ids.ctypes.data, pool.ctypes.data, B, out.ctypes.data, None, None, None) == 0
    print(fake.fake_log().decode(), end="")
""")
    assert [g["threads"] for g in got] == ([threads] * 4 if threads else [1024, 1024, 512, 512])


@pytest.mark.parametrize("H,W", [(64, 64), (72, 104), (8, 8)])
def test_diagnostics_describe_the_request_as_it_is_drawn(fake, H, W):
    got = _launches(fake, f"""
r = bps.bps_create(max_batch=300, height={H}, width={W})
hs = load(r, small), load(r, large)
for B in (1, 9, 17, 40, 300):
    for h in hs:
        for diagnostics in (0, 1, 4):
            bps.bps_set_diagnostics(r, diagnostics)
            ids = np.full(B, h, np.int32)
            fake.fake_clear_log()
            assert lib.bps_render(r, ids.ctypes.data, pool.ctypes.data, B, out.ctypes.data, None, None, None) == 0
            print([l for l in fake.fake_log().decode().splitlines() if l.startswith("k_raster")][0],
                  "said=%d reported=%d" % (bps.bps_query(r, h, 6), bps.bps_query(r, h, 7)))
""")
    assert len(got) == 30 and {g["threads"] for g in got} == {512, 1024}
    for k in range(0, 30, 3):
        for g in got[k:k + 3]:
            assert g["wrong"] == 0 and g["said"] == g["threads"] and g["reported"] == g["lds"]
            assert all(g[x] == got[k][x] for x in ("groups", "tiles", "threads"))


@pytest.mark.parametrize("H,W", [(64, 64), (72, 104), (8, 8)])
def test_reported_lds_is_what_launches_ask_for(fake, H, W):
    p = _launches(fake, f"""
for kw in (dict(), dict(threads=256), dict(threads=1024), dict(splits=2), dict(flags=bps.FLAG_NO_CLUSTER_CULL), dict(flags=bps.FLAG_NO_OCCLUSION_CULL)):
    for diagnostics in (0, 1):
        r = bps.bps_create(max_batch=4, height={H}, width={W}, **kw)
        h = load(r, small)
        bps.bps_set_diagnostics(r, diagnostics)
        ids = np.full(4, h, np.int32)
        fake.fake_clear_log()
        assert lib.bps_render(r, ids.ctypes.data, pool.ctypes.data, 4, out.ctypes.data, None, None, None) == 0
        print([l for l in fake.fake_log().decode().splitlines() if l.startswith("k_raster")][0], "reported=%d" % bps.bps_query(r, h, 7))
""")
    assert len(p) == 12 and all(g["lds"] == g["reported"] for g in p), p
