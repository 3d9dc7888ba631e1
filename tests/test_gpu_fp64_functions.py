"""The FP64 functions of the edge terms against extended precision.

Each is stated to be within 3 units in the last place over its domain
(em_fmath.h).  The reference is numpy's long double (64 bits of mantissa), whose
own error is below 0.01 of a double's unit.  Arguments: all exponents of the
domain, and the neighbourhoods of the points where a form changes range.
"""
import ctypes
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
N = 1 << 20
DIV, SQRT, ATAN2, LOG1P = range(4)


def run(fn, a, b=None):
    import torch

    lib = ctypes.CDLL(os.path.join(ROOT, "paper_2404_17084_amd", "_build", "libemcalib.so"))
    lib.em_calib_fp64.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_void_p] * 3
    x = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    y = torch.from_numpy(np.ascontiguousarray(a if b is None else b)).cuda()
    out = torch.empty_like(x)
    torch.cuda.synchronize()
    assert lib.em_calib_fp64(fn, x.numel(), x.data_ptr(), y.data_ptr(), out.data_ptr()) == 0
    return out.cpu().numpy()


def ulps(got, ref):
    """Largest error in units in the last place of the reference (long double, in a double's range)."""
    d = ref.astype(np.float64)
    return float((np.abs(got.astype(np.longdouble) - ref) / np.spacing(np.abs(d))).max())


def wide(rng, lo, hi, n=N):
    return np.ldexp(rng.uniform(0.5, 1.0, n), rng.integers(lo, hi, n))


def near(rng, at, n=N):
    return at * (1.0 + rng.uniform(-1, 1, n) * np.exp2(-rng.uniform(1, 52, n)))


@pytest.mark.parametrize("lo,hi", [(-60, 60), (-400, 400)])
def test_division(lo, hi):
    rng = np.random.default_rng(1)
    n, d = wide(rng, lo, hi) * rng.choice([-1.0, 1.0], N), wide(rng, lo, hi)
    e = ulps(run(DIV, n, d), n.astype(np.longdouble) / d.astype(np.longdouble))
    print(f"division 2^{lo} to 2^{hi}: {e:.3f}", flush=True)
    assert e < 3.0


@pytest.mark.parametrize("lo,hi", [(-60, 60), (-1000, 1000)])
def test_square_root(lo, hi):
    x = wide(np.random.default_rng(2), lo, hi)
    e = ulps(run(SQRT, x), np.sqrt(x.astype(np.longdouble)))
    print(f"square root 2^{lo} to 2^{hi}: {e:.3f}", flush=True)
    assert e < 3.0


def test_square_root_special_values():
    x = np.array([0.0, -0.0, np.inf, np.nan, -1.0, -np.inf])
    r = run(SQRT, x)
    assert np.array_equal(r[:3], [0.0, 0.0, np.inf]) and np.signbit(r[1]) and np.isnan(r[3:]).all()


@pytest.mark.parametrize("kind", ["any", "tan(pi/8)", "tan(3 pi/8)", "one", "small angles", "near pi", "tiny", "huge"])
def test_arctangent(kind):
    rng = np.random.default_rng(3)
    x = wide(rng, -60, 60) * rng.choice([-1.0, 1.0], N)
    y = np.abs(x) * wide(rng, -30, 30)
    if kind == "tan(pi/8)":
        y = np.abs(x) * near(rng, np.sqrt(2.0) - 1.0)
    elif kind == "tan(3 pi/8)":
        y = np.abs(x) * near(rng, np.sqrt(2.0) + 1.0)
    elif kind == "one":
        y = np.abs(x) * near(rng, 1.0)
    elif kind in ("small angles", "near pi"):
        x = np.abs(x) * (1.0 if kind == "small angles" else -1.0)
        y = np.abs(x) * wide(rng, -200, -20)
    elif kind == "tiny":
        x, y = np.ldexp(x, -900), np.ldexp(y, -900)
    elif kind == "huge":
        x, y = np.ldexp(x, 900), np.ldexp(y, 900)
    e = ulps(run(ATAN2, y, x), np.arctan2(y.astype(np.longdouble), x.astype(np.longdouble)))
    print(f"arctangent, {kind}: {e:.3f}", flush=True)
    assert e < 3.0


def test_arctangent_on_the_axes():
    r = run(ATAN2, np.array([0.0, 0.0, 0.0, 1.0, 1e-310]), np.array([0.0, 1.0, -1.0, 0.0, 0.0]))
    assert np.array_equal(r, [0.0, 0.0, np.pi, np.pi / 2, np.pi / 2])


@pytest.mark.parametrize("kind", ["any", "small", "large", "sqrt(2)", "powers of two", "far apart"])
def test_logarithm_of_a_ratio(kind):
    rng = np.random.default_rng(4)
    d = wide(rng, -60, 60)
    q = {"any": wide(rng, -20, 20), "small": wide(rng, -200, -10), "large": wide(rng, 10, 200),
         "sqrt(2)": np.abs(near(rng, 2.0 ** 0.5) * np.exp2(rng.integers(0, 9, N)) - 1.0),
         "powers of two": np.abs(near(rng, 1.0) * np.exp2(rng.integers(0, 9, N)) - 1.0),
         "far apart": wide(rng, -900, 900)}[kind]
    n = q * d
    e = ulps(run(LOG1P, n, d), np.log1p(n.astype(np.longdouble) / d.astype(np.longdouble)))
    print(f"logarithm, {kind}: {e:.3f}", flush=True)
    assert e < 3.0
