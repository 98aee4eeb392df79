"""The cluster builder's choice of triangles against the rule written out: cheapest candidate first (fewest new
vertices, then nearest to the seed in the maximum norm, then first listed), 64 vertices and 128 triangles at most; and
the clusters that bps_pack_clusters shows are those that scenes are loaded as."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2103_07013_amd as bps
from test_launch_plans import PRELUDE, ROOT, fake  # noqa: F401  (a fixture)

f32 = np.float32


def _grow(v, tris):
    """For one chunk of at most 2048 triangles that are not connected."""
    T = len(tris)
    origin = np.median(v[tris[np.arange(63) * T // 63, 0]], axis=0) * f32(1 / 64)
    p = v[tris] * f32(1 / 64) - origin
    cen = (p[:, 0] + p[:, 1]) + p[:, 2]                     # relative to a place among the triangles, times 3 / 64
    lo = cen.min(0)
    side = max((cen.max(0) - lo).max(), f32(1e-30))
    along = ((cen[:, 0] - lo[0]) + (cen[:, 1] - lo[1])) + (cen[:, 2] - lo[2])
    code = np.minimum(f32(1073741760), along * (f32(1073741823) / (f32(3) * side))).astype(np.uint32)
    order = sorted(range(T), key=lambda t: (code[t], t))    # seeds: along the diagonal
    q = np.clip((cen - lo) * (f32(1023) / side), f32(0), f32(1023)).astype(np.uint32)
    morton = [sum(((int(q[t, a]) >> b) & 1) << (3 * b + a) for a in range(3) for b in range(10)) for t in range(T)]
    curve = sorted(range(T), key=lambda t: (morton[t], t))
    groups = [curve[k:k + 64] for k in range(0, T, 64)]
    boxes = [(cen[g].min(0), cen[g].max(0)) for g in groups]
    at_vertex = [[] for _ in v]
    for t in range(T):
        for i in tris[t]:
            at_vertex[i].append(t)
    taken, clusters = np.zeros(T, bool), []
    for seed in order:
        if taken[seed]:
            continue
        mine, members, cand = set(), [], []
        here, asked, opened, seen, closed = cen[seed], 0, 0, [], []

        def fresh(t):
            return len(set(int(i) for i in tris[t]) - mine)

        def add(t):
            taken[t] = True
            members.append(t)
            for i in tris[t]:
                if int(i) in mine:
                    continue
                mine.add(int(i))
                for o in at_vertex[i]:
                    if len(cand) < 512 and not taken[o] and o not in cand:
                        cand.append(o)

        def nearest():      # in the groups that are open: six at most for the first two, then only what is open
            nonlocal asked, opened, seen, closed
            asked += 1
            if asked == 1:
                closed = [(max(0, *(b[0] - here), *(here - b[1])), g) for g, b in enumerate(boxes) if not taken[groups[g]].all()]
            seen = [x for x in seen if not taken[x[1]]]
            while closed and not (seen and (asked > 2 or opened >= 6 or min(seen)[0] < min(closed)[0])):
                closed.remove(g := min(closed))
                opened += 1
                seen += [(np.abs(cen[t] - here).max(), t) for t in groups[g[1]] if not taken[t]]
            return min(seen)[1] if seen else None
        add(seed)
        while len(members) < 128:
            best = min(cand, key=lambda t: (fresh(t), np.abs(cen[t] - here).max()), default=None)
            if best is None:
                best = nearest()
            if best is None or len(mine) + fresh(best) > 64:
                break
            add(best)
            if best in cand:
                cand.remove(best)
        clusters.append(members)
    return clusters


def _mesh(kind):
    rng = np.random.default_rng(4)
    if kind == "grid":              # equal distances everywhere
        n = 15
        i = np.arange(n * n).reshape(n, n)
        a, b, c, d = i[:-1, :-1].ravel(), i[:-1, 1:].ravel(), i[1:, :-1].ravel(), i[1:, 1:].ravel()
        v = np.stack([*np.meshgrid(np.arange(n), np.arange(n)), np.zeros((n, n))], 2).reshape(-1, 3)
        return v.astype(f32), np.concatenate([np.stack([a, b, c], 1), np.stack([b, d, c], 1)])
    if kind == "soup":              # nothing connected, some triangles degenerate or repeated
        t = np.arange(600).reshape(-1, 3)
        t[::9, 1] = t[::9, 0]
        return rng.normal(size=(600, 3)).astype(f32), np.concatenate([t, t[::7]])
    t = np.stack([np.zeros(2300, int), np.arange(1, 2301), np.arange(2, 2302)], 1)      # one vertex in every triangle
    t[::50, 2] = t[::50, 1]
    return rng.normal(size=(2302, 3)).astype(f32), t


@pytest.fixture(scope="module")
def pack(tmp_path_factory):
    """The members of the clusters that a mesh in one chunk becomes."""
    d, csrc = tmp_path_factory.mktemp("order"), os.path.join(ROOT, "paper_2103_07013_amd", "csrc")
    (d / "shim.cpp").write_text("""
#include "clusters.h"
extern "C" unsigned pack(const float* v, const unsigned* i, unsigned T, unsigned* tris, unsigned* ids) {
    bps::SceneClusters c(v, i, T, T);
    c.write(nullptr, tris, ids, nullptr, 0);
    return c.count();
}
""")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-pthread", "-shared", "-fPIC", "-I" + csrc, str(d / "shim.cpp"),
                    os.path.join(csrc, "clusters.cpp"), "-o", str(d / "shim.so")], check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))

    def run(v, t):
        v, t = np.ascontiguousarray(v, f32), np.ascontiguousarray(t, np.uint32)
        tris, ids = np.zeros((len(t), 128), np.uint32), np.zeros((len(t), 128), np.uint32)
        n = lib.pack(*(a.ctypes.data_as(ctypes.c_void_p) for a in (v, t)), len(t), *(a.ctypes.data_as(ctypes.c_void_p) for a in (tris, ids)))
        return [tuple(int(x) for x in ids[c, :int(tris[c, 0] >> 24)]) for c in range(n)]
    return run


@pytest.mark.parametrize("kind", ["grid", "soup", "fan"])
def test_clusters_follow_the_rule(pack, kind):
    v, t = _mesh(kind)
    assert sorted(pack(v, t)) == sorted(tuple(m) for m in _grow(v, t))


@pytest.mark.parametrize("mesh", ["small", "large", "synth.make_room_scene(1500)"])      # some chunks, two levels of them, one
def test_packed_clusters_are_those_of_a_loaded_scene(fake, mesh):  # noqa: F811
    p = subprocess.run([sys.executable, "-c", PRELUDE + f"""
s = {mesh}
r = bps.bps_create(max_batch=1)
h = load(r, s)
static(r, h, 1)
fake.fake_scenes.restype = ctypes.c_void_p
dev = ctypes.cast(fake.fake_scenes(), ctypes.POINTER(ctypes.c_void_p))      # the scene's record starts with its arrays
for got, k, typ in zip(bps.bps_pack_clusters(s.vertices, s.indices), range(3), (ctypes.c_float, ctypes.c_uint32, ctypes.c_uint32)):
    assert len(got) == bps.bps_query(r, h, 0)
    there = np.ctypeslib.as_array(ctypes.cast(dev[k], ctypes.POINTER(typ)), got.shape)
    assert np.array_equal(got, there)
print("the same")
""", fake], cwd=ROOT, capture_output=True, text=True, timeout=300)
    assert p.returncode == 0 and "the same" in p.stdout, p.stdout + p.stderr


@pytest.mark.parametrize("T", [300, 30_000])
def test_coordinates_that_are_not_finite_are_packed_too(T):
    """bps_load_scene refuses them, bps_pack_clusters does not."""
    rng = np.random.default_rng(8)
    v = rng.normal(size=(T, 3)).astype(f32)
    v[rng.integers(0, T, T // 3), rng.integers(0, 3, T // 3)] = rng.choice([np.nan, np.inf, -np.inf], T // 3)
    _, tris, ids = bps.bps_pack_clusters(v, rng.integers(0, T, (T, 3)).astype(np.uint32))
    assert np.array_equal(np.sort(ids[np.arange(128) < (tris[:, :1] >> 24)]), np.arange(T))
