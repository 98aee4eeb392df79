"""The vertex transform on the matrix cores gives the bits of the one by fmaf, which the numeric rule is stated in: ordinary
numbers, denormal ones, exponents far apart, infinities, and sums that cancel.  (NaNs are equal whatever they carry.)"""
import ctypes
import os

import numpy as np
import pytest

from paper_2103_07013_amd import build as hip

pytestmark = pytest.mark.gpu
HERE = os.path.dirname(os.path.abspath(__file__))
SRC, LIB = os.path.join(HERE, "transforms.hip"), os.path.join(HERE, "libtransforms.so")


def build(force=True):
    if force or not os.path.exists(LIB):
        hip.compile_hip([SRC], LIB)
    return LIB


def bits(rng, shape, exponents):
    """Random signs and mantissas, exponent fields drawn from `exponents`."""
    e = rng.choice(np.asarray(exponents, np.uint32), shape)
    return (rng.integers(0, 2, shape, np.uint32) << 31 | e << 23 | rng.integers(0, 1 << 23, shape, np.uint32)).view(np.float32)


def _inputs(kind, rng, n):
    if kind == "ordinary":
        return rng.normal(size=16).astype(np.float32), (rng.normal(size=(n, 3)) * 10).astype(np.float32)
    if kind == "denormal":      # products, sums and operands at and below the smallest normal number
        return bits(rng, 16, [0, 1, 60, 64, 70]), bits(rng, (n, 3), [0, 1, 2, 55, 60, 66, 70])
    if kind == "mixed exponents":
        return bits(rng, 16, range(0, 255)), bits(rng, (n, 3), range(0, 255))
    if kind == "infinite":      # infinities and NaNs given, and overflows on the way
        p = bits(rng, (n, 3), [1, 127, 253, 254])
        at = rng.random((n, 3)) < .05
        p[at] = rng.choice(np.array([np.inf, -np.inf, np.nan, 0.0, -0.0], np.float32), int(at.sum()))
        return bits(rng, 16, [100, 127, 130, 254]), p
    M = bits(rng, 16, [126, 127])      # cancelling: y and z undo x and the last column to within their rounding
    p = bits(rng, (n, 3), [127, 128])
    p[:, 1] = -(M[0] * p[:, 0]) / M[1] * (1 + rng.integers(-2, 3, n) * 2.0 ** -24)
    p[:, 2] = -(M[3] / M[2]) * (1 + rng.integers(-2, 3, n) * 2.0 ** -24)
    return M, p.astype(np.float32)


@pytest.mark.parametrize("kind", ["ordinary", "denormal", "mixed exponents", "infinite", "cancelling"])
def test_transforms_are_the_same_bits(kind):
    import torch
    lib = ctypes.CDLL(build(force=False))
    n, differ, special = 1 << 16, 0, 0
    out = torch.empty((2, n, 4), dtype=torch.float32, device="cuda")
    for seed in range(16):
        M, p = _inputs(kind, np.random.default_rng([seed, len(kind)]), n)
        M, p = torch.from_numpy(M).cuda(), torch.from_numpy(np.ascontiguousarray(p)).cuda()
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        assert lib.transforms(ctypes.c_void_p(M.data_ptr()), ctypes.c_void_p(p.data_ptr()), n, ctypes.c_void_p(out[0].data_ptr()),
                              ctypes.c_void_p(out[1].data_ptr()), stream) == 0
        torch.cuda.synchronize()
        a, b = out.cpu().numpy()
        same = (a.view(np.uint32) == b.view(np.uint32)) | (np.isnan(a) & np.isnan(b))
        differ += int((~same).sum())
        with np.errstate(invalid="ignore"):
            special += int(((b != 0) & (np.abs(b) < 2.0 ** -126)).sum() if kind == "denormal" else (~np.isfinite(b)).sum() if kind == "infinite" else 1)
    assert differ == 0
    assert special > 0
