"""The error bound under which the threshold-first search proves its results, on the CPU:
scores, norms, bounds and direct distances as the kernels take them (FP16 pairs, a
rounding per matrix instruction of 32 products, FP32 sums lane by lane), on rows whose
roundings all go one way.  The bound's constants come from the library's own header."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1702_08734_amd", "csrc")
SHIM = r"""
#include "sieve_plan.hpp"
extern "C" float err(int dp) { return mk::split_err(dp); }
extern "C" float direct_err() { return mk::kDirectErr; }
"""
f32, f64 = np.float32, np.float64


@pytest.fixture(scope="module")
def bounds(tmp_path_factory):
    d = tmp_path_factory.mktemp("bound")
    (d / "b.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "b.cpp"), "-o",
                    str(d / "b.so")], check=True)
    lib = ctypes.CDLL(str(d / "b.so"))
    lib.err.restype = lib.direct_err.restype = ctypes.c_float
    return lib


def split(v):
    h = v.astype(np.float16)
    return h.astype(f64), (v - h.astype(f32)).astype(np.float16).astype(f64)


def product(x, y):
    """Chain of matrix instructions over 32 components each: h l, l h, h h."""
    (xh, xl), (yh, yl) = split(x), split(y)
    acc = np.zeros(len(x), f32)
    for t in range(0, x.shape[1], 32):
        s = slice(t, t + 32)
        for a, b in ((yh, xl), (yl, xh), (yh, xh)):
            acc = (acc.astype(f64) + (a[:, s] * b[:, s]).sum(1)).astype(f32)
    return acc


def fma_chain(cols):
    s = np.zeros(len(cols), f32)
    for t in range(cols.shape[1]):
        s = (cols[:, t].astype(f64) ** 2 + s).astype(f32)
    return s


def tree(lanes):
    while len(lanes) > 1:
        n = len(lanes) // 2
        lanes = [a + b for a, b in zip(lanes[:n], lanes[n:])]
    return lanes[0]


def norm(v):
    """8 components per granule, granules over up to 16 lanes, a sum over the lanes."""
    g = v.shape[1] // 8
    n = 16 if g > 8 else g
    lanes = []
    for l in range(n):
        at = [8 * (l + n * i) + e for i in range(-(-g // n)) if l + n * i < g for e in range(8)]
        lanes.append(fma_chain(v[:, at]) if at else np.zeros(len(v), f32))
    return tree(lanes)


def direct(x, y):
    """16 lanes of every 16th group of four components."""
    d = x - y
    lanes = [fma_chain(d[:, [t + e for t in range(4 * l, d.shape[1], 64) for e in range(4)]])
             if 4 * l < d.shape[1] else np.zeros(len(d), f32) for l in range(16)]
    return tree(lanes)


def row_bounds(x, y, center, err, direct_err):
    vx, vy = x - center, y - center
    nx, off = norm(vx), norm(vy) * (f32(1) - err)
    score = (product(vx, vy).astype(f64) * -2 + off).astype(f32)
    return (nx * (f32(1) - err) + score) * (f32(1) - direct_err)


# rows of few different components, in [1, 2) and its square root's sizes, beside rows as
# near to them as the distances that a proof is about; with and without a center
@pytest.mark.parametrize("dp", [32, 64, 96, 128, 256])
@pytest.mark.parametrize("values", [1, 2, 8, 1000])
def test_bound_holds(bounds, dp, values):
    rng = np.random.default_rng(dp + values)
    n = 6000
    err, derr = f32(bounds.err(dp)), f32(bounds.direct_err())
    pick = np.arange(dp) % values
    x = (1 + rng.random((n, min(values, dp)))).astype(f32)[:, pick % min(values, dp)]
    for near in (2.0, 1e-1, 1e-3, 1e-5):
        y = (x * (1 + near * (rng.random((n, min(values, dp)))[:, pick % min(values, dp)] - 0.5))).astype(f32)
        for center in (f32(0), f32(0.75), f32(-3.3)):
            low, dist = row_bounds(x, y, center, err, derr), direct(x, y)
            # (a bound below zero proves nothing; the direct form errs too)
            assert (low <= dist).all(), (near, center, (low - dist).max())
