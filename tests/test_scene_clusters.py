"""The clusters a scene is loaded as: every triangle in exactly one of them, within the limits, whatever the mesh and the
number of chunks it is cut into.  clusters.cpp is compiled by itself: no GPU is needed."""
import ctypes
import os
import subprocess
import threading
import time

import numpy as np
import pytest

import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "clusters.h"
extern "C" unsigned pack(const float* v, const unsigned* i, unsigned T, unsigned chunk, unsigned room, float* verts, unsigned* tris,
                         unsigned* ids, float* bounds) {
    bps::SceneClusters c(v, i, T, chunk);
    if (c.count() <= room) c.write(verts, tris, ids, bounds, room);
    return c.count();
}
extern "C" unsigned chunk(unsigned T, int waits) { return bps::chunk_triangles(T, waits != 0); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("clusters")
    (d / "shim.cpp").write_text(SHIM)
    csrc = os.path.join(ROOT, "paper_2103_07013_amd", "csrc")
    subprocess.run(["g++", "-O2", "-std=c++17", "-pthread", "-shared", "-fPIC", "-I" + csrc, str(d / "shim.cpp"),
                    os.path.join(csrc, "clusters.cpp"), "-o", str(d / "shim.so")], check=True)
    return ctypes.CDLL(str(d / "shim.so"))


def _pack(lib, v, t, chunk):
    T, room = len(t), len(t) // 21 + 64 + 2 * (len(t) // chunk)      # a cluster that is full holds 21 triangles or more
    verts, tris = np.zeros((room, 3, 64), np.float32), np.zeros((room, 128), np.uint32)
    ids, bounds = np.zeros((room, 128), np.uint32), np.zeros((6, room), np.float32)
    p = [a.ctypes.data_as(ctypes.c_void_p) for a in (v, t, verts, tris, ids, bounds)]
    C = lib.pack(p[0], p[1], T, chunk, room, *p[2:])
    assert 0 < C <= room
    return verts[:C], tris[:C], ids[:C], bounds[:, :C]


def _mesh(kind):
    rng = np.random.default_rng(11)
    if kind == "scan":
        s = synth.make_multiroom_scene(20_000, seed=5, jitter=0.3)
        return s.vertices, s.indices
    if kind == "soup":              # nothing connected; degenerate and repeated triangles
        t = np.arange(9000).reshape(-1, 3)
        t[::9, 1] = t[::9, 0]
        return rng.normal(size=(9000, 3)), np.concatenate([t, t[::7]])
    if kind == "fan":               # one vertex in every triangle
        return rng.normal(size=(6002, 3)), np.stack([np.zeros(6000, int), np.arange(1, 6001), np.arange(2, 6002)], 1)
    if kind == "point":             # no extent at all
        return np.full((500, 3), 7.0), rng.integers(0, 500, size=(3000, 3))
    if kind == "plane":             # no extent along two axes, and everything on two steps of the third
        return np.stack([rng.integers(0, 2, 2000), np.zeros(2000), np.zeros(2000)], 1), rng.integers(0, 2000, size=(4000, 3))
    if kind == "huge":              # differences of coordinates overflow
        return rng.choice([-3.4e38, 3.4e38, 0.0, 1.0], size=(2000, 3)), rng.integers(0, 2000, size=(4000, 3))
    return np.eye(3), np.array([[0, 1, 2]])


@pytest.mark.parametrize("chunk", [100, 1500, 1 << 20])      # many chunks (two levels of cuts), a few, one
@pytest.mark.parametrize("kind", ["scan", "soup", "fan", "point", "plane", "huge", "one"])
def test_every_triangle_is_in_one_cluster(lib, kind, chunk):
    v, t = (np.ascontiguousarray(a, d) for a, d in zip(_mesh(kind), (np.float32, np.uint32)))
    verts, tris, ids, bounds = _pack(lib, v, t, chunk)
    n = tris[:, 0] >> 24
    used = np.arange(128)[None, :] < n[:, None]
    assert (n >= 1).all() and (n <= 128).all() and (ids[~used] == 0xFFFFFFFF).all() and (tris[~used] == 0).all()
    assert np.array_equal(np.sort(ids[used]), np.arange(len(t)))
    c = np.nonzero(used)[0]
    for k in range(3):
        corner = verts[c, :, (tris[used] >> (8 * k)) & (0xFF if k < 2 else 0x3F)]      # (the top byte of word 0 is the count)
        assert np.array_equal(corner, v[t[ids[used], k]])
    assert np.array_equal(bounds[:3], verts.min(2).T) and np.array_equal(bounds[3:], verts.max(2).T)
    again = _pack(lib, v, t, chunk)      # whichever thread takes which chunk
    assert all(np.array_equal(a, b) for a, b in zip(again, (verts, tris, ids, bounds)))


def _faces(bounds):
    """Sum of the faces of all boxes, as the renderer's tests see them."""
    d = bounds[3:].astype(np.float64) - bounds[:3]
    return (d[0] * d[1] + d[1] * d[2] + d[2] * d[0]).sum()


@pytest.mark.parametrize("far", [-1e30, -1e8, 1e8, 1e30])
def test_a_vertex_that_no_triangle_uses_changes_nothing(lib, far):
    v, t = (np.ascontiguousarray(a, d) for a, d in zip(_mesh("scan"), (np.float32, np.uint32)))
    for chunk in (1500, 1 << 20):
        a, b = _pack(lib, v, t, chunk), _pack(lib, np.concatenate([v, np.full((1, 3), far, np.float32)]), t, chunk)
        assert all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("far", [-1e8, 1e8])
@pytest.mark.parametrize("at", [0, -1])
def test_a_triangle_far_away_leaves_the_others_their_chunks(lib, far, at):
    """Whether it is the first or the last of them.  The clusters are as small as without it, but for its own."""
    v, t = (np.ascontiguousarray(a, d) for a, d in zip(_mesh("scan"), (np.float32, np.uint32)))
    clean = _pack(lib, v, t, 1500)
    more = np.array([[far, 0, 0], [far, 1e3, 0], [far, 0, 1e3]], np.float32)
    t2 = np.insert(t, 0 if at == 0 else len(t), np.arange(len(v), len(v) + 3, dtype=np.uint32), axis=0)
    _, _, ids, bounds = _pack(lib, np.concatenate([v, more]), t2, 1500)
    rest = bounds[:, ~(ids == (0 if at == 0 else len(t))).any(1)]
    assert _faces(rest) < 1.1 * _faces(clean[3]) and rest.shape[1] < 1.1 * clean[3].shape[1]


@pytest.mark.parametrize("place", ["spread", "one"])
def test_loose_triangles_take_time_in_proportion(lib, place):
    """No two connected, in one chunk: four times as many take about four times as long (where every cluster looks at
    all groups of the chunk, nine times or more; seven lies between)."""
    def best(n):
        rng = np.random.default_rng(5)
        c = rng.uniform(-5, 5, (n if place == "spread" else 1, 1, 3))
        v = np.ascontiguousarray(np.resize(c + rng.normal(0, 0.03, (len(c), 3, 3)), (3 * n, 3)), np.float32)
        t = np.arange(3 * n, dtype=np.uint32).reshape(-1, 3)
        p = [a.ctypes.data_as(ctypes.c_void_p) for a in (v, t)]
        times = []
        for _ in range(3):
            t0 = time.thread_time()      # (the chunk is grown by the calling thread; others' load does not count)
            lib.pack(*p, n, 1 << 20, 0, None, None, None, None)
            times.append(time.thread_time() - t0)
        return min(times)
    assert best(360_000) < 7 * best(90_000)


@pytest.mark.parametrize("cpus", [1, 2])
def test_no_more_threads_than_cpus_the_caller_may_use(lib, cpus):
    """A loader keeps its scenes' packing to some CPUs by its own affinity mask."""
    mine = sorted(os.sched_getaffinity(0))
    if len(mine) < 4:
        pytest.skip("too few CPUs to tell")
    v, t = (np.ascontiguousarray(a, d) for a, d in zip(_mesh("scan"), (np.float32, np.uint32)))
    t = np.ascontiguousarray(np.resize(t, (600_000, 3)))
    p = [a.ctypes.data_as(ctypes.c_void_p) for a in (v, t)]

    def most(mask):
        def load():
            os.sched_setaffinity(0, mask)      # (of this thread alone)
            lib.pack(*p, len(t), 16384, 0, None, None, None, None)
        before, th, seen = len(os.listdir("/proc/self/task")), threading.Thread(target=load), 0
        th.start()
        while th.is_alive():
            seen = max(seen, len(os.listdir("/proc/self/task")))
        th.join()
        return seen - before
    assert most(mine[:cpus]) <= cpus and 2 < most(mine) <= 12


def test_chunks_are_neither_empty_nor_too_many(lib):
    """From 6144 triangles on there is work for a second thread, whether the caller waits for the scene or not."""
    for T in [1, 2, 4999, 6143, 6144, 9_999, 20_000, 32_767, 32_768, 65_535, 65_537, 100_000, 200_000, 1_000_000, 0xFFFFFFFF]:
        for waits, most in ((1, 65536), (0, 16384)):
            chunk = lib.chunk(T, waits) & 0xFFFFFFFF
            assert 3073 <= chunk <= most
            n = -(-T // chunk)
            assert n == 1 if T < 6144 else 2 <= n <= max(12, T // most + 1)
