"""What the batch renderer is asked to do in earnest, as a list of cases that can be timed.

A case is one request through the public entry points: a batch of environments, each naming one of K
resident scenes and a camera, in; one low-resolution frame per environment, left in GPU memory, out.
Scenes and cameras are the seeded procedural ones of `synth` (multi-room scans of 10 k to 1 M triangles,
level agent cameras), the shapes and sizes those of the repository's workloads, tests and sweep.

Fields of a case:
  entry      "render" (Renderer.render), "static" (bps_render_static), "rotate" (asynchronous scene load,
             a request that uses the new scene, retirement of the scene)
  scene      "room" or "multiroom"; K scenes of about T triangles; jitter > 0: irregular geometry
  B, H, W    environments and output frame
  mode       "depth", "rgbd" (vertex colours) or "textured"; bilinear, supersample as in bps_config
  ids        the caller wants the winning triangle ids as well
  host_vp    the matrices are host arrays (a CPU simulator hands over poses) instead of device tensors
"""
import math

import numpy as np
import torch

import paper_2103_07013_amd as bps
import synth

_DEFAULTS = dict(entry="render", scene="multiroom", K=1, T=200_000, jitter=0.0, B=256, H=64, W=64, mode="depth",
                 bilinear=False, supersample=1, ids=False, host_vp=False)


def _case(**kw):
    return {**_DEFAULTS, **kw}


def listed():
    return [
        # evaluation of a single agent: the smallest call there is, latency and launches count
        _case(name="single_agent", B=1, ids=True),
        # a handful of environments in one small room (the smoke-test and debugging workload)
        _case(name="room_16", scene="room", T=10_000, B=16, ids=True),
        # a few environments with a wide, odd-sized frame that is no square and no power of two
        _case(name="ragged_61", K=3, T=100_000, B=61, H=72, W=104),
        # one GPU's share of a multi-GPU run: 256 environments in one scan, poses from a CPU simulator
        _case(name="batch_256", B=256, host_vp=True),
        # the paper's main configuration: 1024 environments, four scans, 64x64 depth
        _case(name="batch_1024", K=4, T=500_000, B=1024),
        # the same with geometry as irregular as a real scan, a batch size that is no power of two, host poses
        _case(name="scan_1000", K=4, T=500_000, jitter=0.3, B=1000, host_vp=True),
        # RGB-D agents on large scans
        _case(name="rgbd_1024", K=4, T=1_000_000, B=1024, mode="rgbd"),
        # RGB agents on textured scans, rendered at twice the resolution and averaged down
        _case(name="textured_ss_192", K=2, T=200_000, B=192, mode="textured", bilinear=True, supersample=2),
        # the larger encoder's 128x128 frames at the largest batch
        _case(name="large_4096_128", K=4, T=1_000_000, B=4096, H=128, W=128),
        # the entry point for callers that cannot allocate
        _case(name="static_512", entry="static", K=2, T=200_000, B=512, ids=True),
        # scene rotation: a new scan is streamed in, used by half of a small batch and retired
        _case(name="rotate_64", entry="rotate", K=1, T=100_000, B=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["depth", "depth", "depth", "rgbd", "textured", "static", "rotate"])
    c = dict(K=rng.randint(1, 4), T=_log_int(rng, 10_000, 1_000_000), jitter=rng.choice([0.0, 0.0, 0.3]),
             B=_log_int(rng, 1, 2048))
    side = rng.choice(["64", "64", "128", "any"])
    if side == "any":
        c.update(H=8 * rng.randint(3, 16), W=8 * rng.randint(3, 16))
    else:
        c.update(H=int(side), W=int(side))
    c["ids"] = rng.random() < 0.4
    if kind == "depth":
        c["host_vp"] = rng.random() < 0.4
        if c["T"] < 40_000 and rng.random() < 0.5:
            c.update(scene="room", jitter=0.0)
    elif kind == "static":
        c["entry"] = "static"
    elif kind == "rotate":
        c.update(entry="rotate", T=_log_int(rng, 10_000, 200_000), B=max(2, c["B"] // 4))
    else:
        c["mode"] = kind
        if kind == "textured":
            c["bilinear"] = rng.random() < 0.5
            if c["H"] <= 64 and c["W"] <= 64 and rng.random() < 0.6:
                c.update(supersample=2, ids=False)
    c["K"] = min(c["K"], c["B"])
    return _case(**c)


def _scene(case, seed):
    if case["scene"] == "room":
        return synth.make_room_scene(case["T"], seed=seed)
    return synth.make_multiroom_scene(case["T"], seed=seed, jitter=case["jitter"])


def _load(r, s, mode):
    if mode == "textured":
        return r.load_scene_textured(s.vertices, s.indices, s.uvs, s.texture)
    return r.load_scene(s.vertices, s.indices, s.colors if mode == "rgbd" else None)


def prepare(case, seed):
    """Renderer with its resident scenes, the poses of the step, and the observation buffers."""
    K, B, H, W = case["K"], case["B"], case["H"], case["W"]
    flags = bps.FLAG_BILINEAR if case["bilinear"] else 0
    r = bps.Renderer(max_batch=B, height=H, width=W, mode=bps.MODE_DEPTH if case["mode"] == "depth" else bps.MODE_RGBD,
                     flags=flags, supersample=case["supersample"])
    n_scenes = K + 1 if case["entry"] == "rotate" else K
    scenes = [_scene(case, 1_000_003 * (seed + 1) + k) for k in range(n_scenes)]
    handles = [_load(r, s, case["mode"]) for s in scenes[:K]]
    which = np.arange(B) % n_scenes
    vp = np.empty((B, 4, 4), np.float32)
    for k in range(n_scenes):
        at = np.nonzero(which == k)[0]
        if at.size:
            vp[at] = synth.make_cameras(scenes[k], at.size, seed=7919 * (seed + 1) + k, aspect=W / H)[0]
    dev = torch.device("cuda", 0)
    st = {"case": case, "r": r, "vp": vp if case["host_vp"] else torch.from_numpy(vp).to(dev), "which": which,
          "scene_ids": np.array([handles[w] if w < K else -1 for w in which], np.int32),
          "depth": torch.empty((B, H, W), dtype=torch.float32, device=dev), "rgb": None, "tri": None}
    if case["mode"] != "depth":
        st["rgb"] = torch.empty((B, H, W, 3), dtype=torch.uint8, device=dev)
    if case["ids"]:
        st["tri"] = torch.empty((B, H, W), dtype=torch.int32, device=dev)
    if case["entry"] == "rotate":
        st["new"] = scenes[K]
        st["copy_stream"] = torch.cuda.Stream()
    return st


def run(st):
    """One request; the frames it leaves in GPU memory."""
    r, entry, K = st["r"], st["case"]["entry"], st["case"]["K"]
    if entry == "static":
        bps.bps_render_static(r.handle, st["scene_ids"], st["vp"], st["depth"], st["tri"])
    elif entry == "rotate":
        new = r.load_scene_async(st["new"].vertices, st["new"].indices, copy_stream=st["copy_stream"])
        ids = np.where(st["which"] == K, new, st["scene_ids"]).astype(np.int32)
        r.render(ids, st["vp"], out_depth=st["depth"], out_tri_id=st["tri"])
        r.unload_scene(new)
    else:
        r.render(st["scene_ids"], st["vp"], out_depth=st["depth"], out_rgb=st["rgb"], out_tri_id=st["tri"])
    return [t for t in (st["depth"], st["rgb"], st["tri"]) if t is not None]


def work(case):
    """Every input read once (the scenes' vertices and indices, with V about T / 2; per-vertex colours or
    texture coordinates; the matrices), every output written once.  Operations: per rendered pixel one
    covering triangle's three edge functions, its interpolated 1/w and depth (22), and the transform of
    three vertices (3 x 28); colour adds three interpolated channels (18)."""
    T, V, B = case["T"], case["T"] // 2, case["B"]
    scenes = case["K"] + (1 if case["entry"] == "rotate" else 0)
    mesh = 12 * T + 12 * V
    if case["mode"] == "rgbd":
        mesh += 3 * V
    elif case["mode"] == "textured":
        mesh += 8 * V + 256 * 256 * 3
    pixels = B * case["H"] * case["W"]
    out = 4 + (0 if case["mode"] == "depth" else 3) + (4 if case["ids"] else 0)
    samples = pixels * case["supersample"] ** 2
    return {"bytes": scenes * mesh + 64 * B + pixels * out,
            "flops": samples * (22 + 84 + (0 if case["mode"] == "depth" else 18))}


def tolerance(case):
    """The numeric rule fixes every float operation and its order (see include/bps.h and the oracle), and the
    frame is the minimum of integer keys, so any correct implementation gives the same bits."""
    return "exact"
