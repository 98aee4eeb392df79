"""Scene loads, requests and retirements that find no memory, without a GPU (fake_hip.c): they end as an error, whichever
allocation it was that failed, and leave nothing behind."""
import subprocess
import sys

import pytest

from test_launch_plans import PRELUDE, ROOT, fake  # noqa: F401  (a fixture)

# an operator new that fails once, when the countdown has run out; libbps.so finds it before the usual one
FAILING_NEW = """
#include <atomic>
#include <cstdlib>
#include <new>
static std::atomic<long> left{-1};
extern "C" void fail_after(long n) { left = n; }
extern "C" long fail_left() { return left; }
void* operator new(std::size_t n) {
    if (left >= 0 && left-- == 0) throw std::bad_alloc();
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
"""


def _run(fake, code, *args):  # noqa: F811
    p = subprocess.run([sys.executable, "-c", PRELUDE + code, fake, *args], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.endswith("done\n"), p.stdout + p.stderr


def _run_failing(fake, failing_new, code):  # noqa: F811
    """With `new` as the library of that operator, loaded before libbps.so (which the prelude loads)."""
    code = PRELUDE.replace("import paper_2103_07013_amd", "new = ctypes.CDLL(sys.argv[2], mode=ctypes.RTLD_GLOBAL)\nnew.fail_left.restype = ctypes.c_long\n"
                           "import paper_2103_07013_amd", 1) + code
    p = subprocess.run([sys.executable, "-c", code, fake, failing_new], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and p.stdout.endswith("done\n"), p.stdout + p.stderr


@pytest.fixture(scope="module")
def failing_new(tmp_path_factory):
    d = tmp_path_factory.mktemp("new")
    (d / "new.cpp").write_text(FAILING_NEW)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "new.cpp"), "-o", str(d / "new.so")], check=True)
    return str(d / "new.so")


@pytest.mark.parametrize("T,step", [(600, 1), (8000, 3)])      # one thread, and two
def test_any_allocation_of_a_load_may_fail(fake, failing_new, T, step):  # noqa: F811
    _run_failing(fake, failing_new, f"""
s = synth.make_room_scene({T})
v, t = np.ascontiguousarray(s.vertices, np.float32), np.ascontiguousarray(s.indices, np.uint32)
r = bps.bps_create(max_batch=1)
def attempt(n):
    h = ctypes.c_int32(-1)
    new.fail_after(ctypes.c_long(n))
    st = lib.bps_load_scene(r, v.ctypes.data, len(v), t.ctypes.data, len(t), None, ctypes.byref(h))
    left = new.fail_left()
    new.fail_after(ctypes.c_long(-1))
    assert st in (0, -3), st
    if st == 0:
        assert lib.bps_unload_scene(r, h) == 0
    return st, left
n = failures = 0
while True:
    st, left = attempt(n)
    failures += st == -3
    if left >= 0:      # there was none left to fail
        break
    n += {step}
assert st == 0 and failures > 20, (failures, n)
assert fake.fake_live(1) == 1 and fake.fake_allocated(1) == 1, "one pinned image served all of them"
assert bps.bps_query(r, 0, 8) == 1, "and so did one device block"
bps.bps_destroy(r)
assert fake.fake_live(0) == fake.fake_live(1) == 0
print("done")
""")


def test_any_allocation_of_a_request_or_a_retirement_may_fail(fake, failing_new):  # noqa: F811
    """Each call is made again until it succeeds, with another allocation failing every time; what is drawn then is right."""
    _run_failing(fake, failing_new, """
r = bps.bps_create(max_batch=300)
def until_it_succeeds(call):
    for n in range(100):
        new.fail_after(ctypes.c_long(n))
        st = call()
        new.fail_after(ctypes.c_long(-1))
        assert st in (0, -3), st
        if st == 0:
            return n
    raise SystemExit("never")
failures = 0
bps.bps_set_profiling(r, 1)
for B in (300, 17, 300, 5):
    h = load(r, small if B == 17 else large)
    ids = np.full(B, h, np.int32)
    for k in range(2):
        fake.fake_clear_log()
        failures += until_it_succeeds(lambda: lib.bps_render(r, ids.ctypes.data, pool.ctypes.data, B, out.ctypes.data, None, None, None))
        failures += until_it_succeeds(lambda: lib.bps_render_static(r, ids.ctypes.data, pool.ctypes.data, B, out.ctypes.data, None, None))
        drawn = [l for l in fake.fake_log().decode().splitlines() if l.startswith("k_raster")]
        assert len(drawn) == 2 and all(f" envs={B} " in l and " wrong=0 " in l for l in drawn), drawn
    failures += until_it_succeeds(lambda: lib.bps_unload_scene(r, h))
assert failures > 20, failures
print("done")
""")


def test_no_room_for_the_pinned_image_or_the_device_block(fake):  # noqa: F811
    _run(fake, """
r = bps.bps_create(max_batch=1)
for pinned in (1, 0):
    fake.fake_largest(pinned, ctypes.c_size_t(10_000))
    for _ in range(3):
        try:
            load(r, small)
            raise SystemExit("loaded")
        except bps.BpsError as e:
            assert e.status == -3, e
    fake.fake_largest(pinned, ctypes.c_size_t(1 << 40))
a, b = load(r, small), load(r, small)
bps.bps_unload_scene(r, a)
load(r, small)
assert fake.fake_live(1) == 1 and bps.bps_query(r, 0, 8) == 2
print("done")
""")


def test_a_device_block_is_as_large_as_the_scene_where_there_is_no_more(fake):  # noqa: F811
    """Blocks come in coarse sizes, which must not refuse a scene that fits."""
    _run(fake, """
r = bps.bps_create(max_batch=1)
scenes = [synth.make_room_scene(T) for T in (300, 3000, 10_000)] + [small, large]
for s in scenes:
    h = load(r, s)
    coarse = fake.fake_last_size(0)
    fake.fake_largest(0, ctypes.c_size_t(coarse - 1))
    g = load(r, s)
    exact = fake.fake_last_size(0)
    assert bps.bps_query(r, h, 3) == coarse and bps.bps_query(r, g, 3) == exact      # what they hold
    assert coarse - max(4096, coarse // 16) <= exact < coarse, (exact, coarse)
    fake.fake_largest(0, ctypes.c_size_t(exact - 1))
    try:
        load(r, s)
        raise SystemExit("loaded")
    except bps.BpsError as e:
        assert e.status == -3, e
    fake.fake_largest(0, ctypes.c_size_t(1 << 40))
print("done")
""")
