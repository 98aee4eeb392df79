"""The event of a request, without a GPU (fake_hip.c in the place of the HIP runtime): every kind of request sets its slot's
event once, with the last thing it enqueues, and what a request reads is not given away before that event is reached."""
import re
import subprocess
import sys

import pytest

from test_launch_plans import PRELUDE, ROOT, fake      # noqa: F401  (a fixture)

SETUP = PRELUDE + """
fake.fake_ops.restype = ctypes.c_char_p
mesh = synth.make_room_scene(1_000, seed=3)
def renderer(B=300, **kw):
    r = bps.bps_create(max_batch=B, **kw)
    h = bps.bps_load_scene(r, mesh.vertices, mesh.indices, mesh.colors)
    return r, h
def render(r, h, B=300, rgb=False, vp=pool):
    ids = np.full(B, h, np.int32)
    st = lib.bps_render(r, ids.ctypes.data, vp.ctypes.data, B, out.ctypes.data, out.ctypes.data if rgb else None, None, None)
    assert st == 0, bps.bps_last_error(r)
def render_static(r, h, B=300):
    ids = np.full(B, h, np.int32)
    st = lib.bps_render_static(r, ids.ctypes.data, pool.ctypes.data, B, out.ctypes.data, None, None)
    assert st == 0, bps.bps_last_error(r)
def ops(call):
    fake.fake_clear_ops()
    call()
    print("request", " | ".join(fake.fake_ops().decode().splitlines()))
"""


def _run(fake, code):
    p = subprocess.run([sys.executable, "-c", SETUP + code, fake], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0, p.stdout + p.stderr
    return p.stdout.splitlines()


def _requests(fake, code):
    """Per request: its operations, each (kernel or "record", event number or None)."""
    out = []
    for line in _run(fake, code):
        if line.startswith("request "):
            out.append([(re.sub(r"^_ZN3bps\d+(k_[a-z_]+?)(I[A-Z].*|E.*)$", r"\1", o.split(" ")[0]), int(o.split("event=")[1]) if "event=" in o else None)
                        for o in line[8:].split(" | ")])
    return out


# kind of request: set-up and call, and what carries the event
KINDS = {
    "depth": ("r, h = renderer()", "render(r, h)", "k_raster"),
    "one environment": ("r, h = renderer(1)", "render(r, h, 1)", "k_raster"),
    "planned ahead": ("r, h = renderer(600); far = np.zeros((600, 16), np.float32)", "render(r, h, 600, vp=far)", "k_raster"),
    "diagnostics": ("r, h = renderer(); bps.bps_set_diagnostics(r, 1)", "render(r, h)", "k_raster"),
    "rgbd": ("r, h = renderer(mode=bps.MODE_RGBD)", "render(r, h, rgb=True)", "k_shade"),
    "rgbd of split frames": ("r, h = renderer(mode=bps.MODE_RGBD, splits=2)", "render(r, h, rgb=True)", "k_shade"),
    "rgbd timed": ("r, h = renderer(mode=bps.MODE_RGBD); bps.bps_set_profiling(r, 1)", "render(r, h, rgb=True)", "k_shade"),
    "supersampled": ("r, h = renderer(supersample=2)", "render(r, h)", "k_downsample"),
    "rgbd supersampled": ("r, h = renderer(mode=bps.MODE_RGBD, supersample=2)", "render(r, h, rgb=True)", "k_downsample"),
    "split": ("r, h = renderer(splits=2)", "render(r, h)", "record"),
    "timed": ("r, h = renderer(); bps.bps_set_profiling(r, 1)", "render(r, h)", "record"),
    "static": ("r, h = renderer()", "render_static(r, h)", "k_raster"),
}


@pytest.mark.parametrize("kind", list(KINDS))
def test_event_is_set_once_by_the_last_operation(fake, kind):      # noqa: F811
    setup, call, last = KINDS[kind]
    got = _requests(fake, f"{setup}\nfor _ in range(9):\n    ops(lambda: {call})\n")
    assert len(got) == 9
    events = [r[-1][1] for r in got]
    assert all(r[-1][0] == last for r in got), got[0]
    assert all(sum(e == r[-1][1] for _, e in r) == 1 for r in got), got
    assert len(set(events[:4])) == 4 and events[4:] == events[:5]      # the four slots in turn


@pytest.mark.parametrize("entry,setup", [("render(r, h)", "renderer()"), ("render(r, h, rgb=True)", "renderer(mode=bps.MODE_RGBD)"),
                                         ("render(r, h)", "renderer(supersample=2)")])
def test_captured_request_records_its_event(fake, entry, setup):      # noqa: F811
    got = _requests(fake, f"""
r, h = {setup}
{entry}
fake.fake_capture(1)
ops(lambda: {entry})
fake.fake_capture(0)
""")
    assert [e for _, e in got[0][:-1]] == [None] * (len(got[0]) - 1) and got[0][-1][0] == "record"


def test_captured_static_request_has_no_event(fake):      # noqa: F811
    got = _requests(fake, """
r, h = renderer()
fake.fake_capture(1)
ops(lambda: render_static(r, h))
fake.fake_capture(0)
""")
    assert all(e is None for _, e in got[0]) and got[0][-1][0] == "k_raster"


@pytest.mark.parametrize("entry", ["render(r, h)", "render_static(r, h)"])
def test_event_is_recorded_where_a_capture_cannot_be_ruled_out(fake, entry):      # noqa: F811
    got = _requests(fake, f"""
r, h = renderer()
fake.fake_capture_unknown(1)
ops(lambda: {entry})
""")
    assert got[0][-1][0] == "record" and all(e is None for _, e in got[0][:-1])


@pytest.mark.parametrize("kind", list(KINDS))
def test_scene_is_kept_until_the_event_is_reached(fake, kind):      # noqa: F811
    setup, call, _ = KINDS[kind]
    lines = _run(fake, f"""
{setup}
{call}
fake.fake_hold(1)
{call}
bps.bps_unload_scene(r, h)
a = bps.bps_query(r, 0, 8)
load = lambda: bps.bps_load_scene(r, mesh.vertices, mesh.indices, mesh.colors)
other = load()
b = bps.bps_query(r, 0, 8)
fake.fake_hold(0)
third = load()
print("blocks", a, b, bps.bps_query(r, 0, 8))
""")
    a, b, c = map(int, lines[-1].split()[1:])
    assert b == a + 1 and c == b      # held: a block of its own; reached: the retired one
