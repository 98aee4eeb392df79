"""The cluster builder's choice of triangles against the rule written out: cheapest candidate first (fewest new
vertices, then nearest to the seed in the maximum norm, then first listed), 64 vertices and 128 triangles at most."""
import numpy as np
import pytest

import paper_2103_07013_amd as bps

f32 = np.float32


def _grow(v, tris):
    T = len(tris)
    cen = ((v[tris[:, 0]] + v[tris[:, 1]]) + v[tris[:, 2]]) * f32(1.0 / 3.0)
    lo = v.min(0)
    scale = f32(1023.0) / max((v.max(0) - lo).max(), f32(1e-20))
    q = np.clip((cen - lo) * scale, f32(0), f32(1023)).astype(np.uint32)
    code = [sum(((int(q[t, a]) >> b) & 1) << (3 * b + a) for a in range(3) for b in range(10)) for t in range(T)]
    order = sorted(range(T), key=lambda t: (code[t], t))
    at_vertex = [[] for _ in v]
    for t in range(T):
        for i in tris[t]:
            at_vertex[i].append(t)
    taken, clusters = np.zeros(T, bool), []
    for seed in order:
        if taken[seed]:
            continue
        mine, members, cand = set(), [], []

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
        add(seed)
        while len(members) < 128:
            best = min(cand, key=lambda t: (fresh(t), np.abs(cen[t] - cen[seed]).max()), default=None)
            if best is None:      # nothing connected: the first of the next 192 in order that brings in the fewest
                best = min([t for t in order if not taken[t]][:192], key=fresh, default=None)
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


@pytest.mark.parametrize("kind", ["grid", "soup", "fan"])
def test_clusters_follow_the_rule(kind):
    v, t = _mesh(kind)
    _, tris, ids = bps.bps_pack_clusters(v, t.astype(np.uint32))
    got = sorted(tuple(int(x) for x in ids[c, :int(tris[c, 0] >> 24)]) for c in range(len(ids)))
    assert got == sorted(tuple(m) for m in _grow(v, t))
