"""The FP64 arctangent and reciprocal root of the kernels (rir_device.h,
atan2_abs and d_rsqrt) against their stated error bounds, on the CPU: the same
steps in 80-bit extended precision, rounded to FP64 where the kernels round, with
hardware estimates off by up to 2^-23 of their value either way.  The table is
read from the header."""
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2112_02779_amd", "csrc", "rir_device.h")
LD = np.longdouble

pytestmark = pytest.mark.skipif(np.finfo(LD).nmant < 63, reason="needs 80-bit extended precision")


def _fma(a, b, c):
    """One rounding to FP64 (the product's rounding to 64 bits before it moves
    the result by far less than the bounds tested)."""
    return (np.asarray(a, LD) * np.asarray(b, LD) + np.asarray(c, LD)).astype(np.float64)


def _estimate(x, off):
    return (np.asarray(x, LD) * (1 + LD(off))).astype(np.float64)


def _table():
    text = open(HEADER).read()
    body = text[text.index("kAtan16[17] = {"):]
    return np.array([float(v) for v in body[body.index("{") + 1:body.index("}")].split(",")])


def _atan2_abs(y, x, off):
    T = _table()
    ax, ay = np.abs(x), np.abs(y)
    mx, mn = np.maximum(np.maximum(ax, ay), 1e-290), np.minimum(ax, ay)
    k = np.rint(16.0 * mn * _estimate(1 / mx.astype(LD), off))
    ki = np.minimum(k.astype(np.int64), 16)
    c = 0.0625 * k
    num, den = _fma(-c, mx, mn), _fma(c, mn, mx)
    inv = _estimate(1 / den.astype(LD), off)
    e = _fma(-den, inv, 1.0)
    inv = _fma(inv, _fma(e, e, e), inv)
    t = num * inv
    t = _fma(_fma(-den, t, num), inv, t)
    t2 = t * t
    p = _fma(t2, 1.0 / 9.0, -1.0 / 7.0)
    p = _fma(p, t2, 1.0 / 5.0)
    p = _fma(p, t2, -1.0 / 3.0)
    p = _fma(p * t2, t, t) + T[ki]
    hi, lo = 1.57079632679489661923, 6.123233995736766036e-17
    p = np.where(ay > ax, hi - (p - lo), p)
    return np.where(x < 0, 2 * hi - (p - 2 * lo), p)


def test_table_entries():
    T = _table()
    assert T.size == 17
    np.testing.assert_array_equal(T, np.arctan(np.arange(17, dtype=LD) / 16).astype(np.float64))


@pytest.mark.parametrize("off", [0.0, 2.0 ** -23, -2.0 ** -23])
def test_atan2_within_two_ulps(off):
    rng = np.random.default_rng(1)
    n = 400_000
    a = rng.uniform(-np.pi, np.pi, n)
    r = np.exp(rng.uniform(np.log(1e-6), np.log(1e6), n))
    x, y = r * np.cos(a), r * np.sin(a)
    # quotients at and next to the table's edges, both sides of a diagonal, axes
    q = np.concatenate([np.nextafter((2 * np.arange(16) + 1) / 32, d) for d in (0.0, 2.0)] +
                       [np.arange(17) / 16, 10.0 ** -np.arange(1, 17)])
    x = np.concatenate([x, np.ones_like(q), q, -np.ones_like(q), -q])
    y = np.concatenate([y, q, np.ones_like(q), q, -np.ones_like(q)])
    got = _atan2_abs(y, x, off)
    ref = np.arctan2(np.abs(y).astype(LD), x.astype(LD))
    err = np.abs(got.astype(LD) - ref) / np.spacing(ref.astype(np.float64))
    assert err.max() < 2.0, float(err.max())


def test_atan2_of_zeros_and_axes():
    z = np.array([0.0])
    assert _atan2_abs(z, z, 0.0)[0] == 0.0
    assert _atan2_abs(z, np.array([2.0]), 0.0)[0] == 0.0
    assert _atan2_abs(z, np.array([-2.0]), 0.0)[0] == np.pi
    assert _atan2_abs(np.array([-3.0]), z, 0.0)[0] == np.pi / 2


@pytest.mark.parametrize("off", [0.0, 2.0 ** -23, -2.0 ** -23])
def test_reciprocal_root_within_one_ulp(off):
    rng = np.random.default_rng(2)
    x = np.exp(rng.uniform(np.log(1e-300), np.log(1e300), 400_000))
    ref = 1 / np.sqrt(x.astype(LD))
    y = _estimate(ref, off)
    h = _fma(-x * y, y, 1.0)
    got = _fma(y * h, _fma(0.375, h, 0.5), y)
    err = np.abs(got.astype(LD) - ref) / np.spacing(ref.astype(np.float64))
    assert err.max() < 1.0, float(err.max())


def test_formulas_are_the_headers():
    """The lines transcribed above are those of the header."""
    text = re.sub(r"\s+", " ", open(HEADER).read())
    for line in ("const double k = rint(16.0 * mn * __builtin_amdgcn_rcp(mx));",
                 "const double num = fma(-c, mx, mn), den = fma(c, mn, mx);", "inv = fma(inv, fma(e, e, e), inv);",
                 "t = fma(fma(-den, t, num), inv, t);", "double p = fma(t2, 1.0 / 9.0, -1.0 / 7.0);",
                 "p = fma(p * t2, t, t) + kAtan16[ki];", "p = ay > ax ? hi - (p - lo) : p;",
                 "return x < 0.0 ? 2.0 * hi - (p - 2.0 * lo) : p;", "const double h = fma(-x * y, y, 1.0);",
                 "return fma(y * h, fma(0.375, h, 0.5), y);"):
        assert line in text, line
