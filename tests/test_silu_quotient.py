"""silu(z) = z / (1 + exp(-z)) in the network kernels (kpsi_silu.h) against the IEEE division, on the CPU:
the quotient is that of the division for every estimate of the reciprocal within one unit in the last
place, and saturated units, infinities and NaN give what the division gives."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "kpsi_silu.h"
extern "C" void run(long n, const float* z, const float* d, const float* y0, float* sl, float* sl2, float* ds) {
  for (long i = 0; i < n; ++i) {
    sl[i] = kpsi::nn::silu_of(z[i], d[i], y0[i]);
    kpsi::nn::silu_both_of(z[i], d[i], y0[i], sl2[i], ds[i]);
  }
}
"""
F = np.float32


@pytest.fixture(scope="module")
def silu(tmp_path_factory):
    from paper_2007_14931_amd import build
    d = tmp_path_factory.mktemp("silu")
    src, lib = d / "shim.hip", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Xclang",
                    "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", build.CSRC, str(src), "-o", str(lib)],
                   check=True, capture_output=True)
    run = ctypes.CDLL(str(lib)).run

    def f(z, d, y0):
        z, d, y0 = (np.ascontiguousarray(x, dtype=F) for x in (z, d, y0))
        out = [np.empty_like(z) for _ in range(3)]
        run(ctypes.c_long(z.size), *(ctypes.c_void_p(x.ctypes.data) for x in (z, d, y0, *out)))
        return out
    return f


def _same(a, b):
    return np.array_equal(a.view(np.uint32), b.view(np.uint32))


def _near_midpoints(rng, n):
    """z and d whose quotient is within 2^-49 of the middle between two floats: m d = c mod 2^25 for the
    odd 25-bit midpoint m and a small odd c, z = (m d - c) / 2^25."""
    d = (rng.integers(2**22, 2**23, n) * 2 + 1).astype(object)
    m = np.array([pow(int(x), -1, 2**25) for x in d], dtype=object) * rng.choice([-3, -1, 1, 3], n) % 2**25
    keep = m >= 2**24
    d, m = d[keep], m[keep]
    z = (m * d + 2**24) // 2**25
    return z.astype(np.float64).astype(F) * F(2.0**-23), d.astype(np.float64).astype(F) * F(2.0**-23)


@pytest.mark.parametrize("ulp", [-1, 0, 1])
def test_quotient_is_the_ieee_quotient(silu, ulp):
    rng = np.random.default_rng(7 + ulp)
    z = rng.choice([-1, 1], 4_000_000) * np.exp(rng.uniform(-12, 4.46, 4_000_000))   # up to |z| = 86
    z = z.astype(F)
    d = (F(1) + np.exp(-z)).astype(F)
    d[::2] = np.nextafter(d[::2], F(2) * d[::2])
    zm, dm = _near_midpoints(rng, 400_000)
    n = z.size
    z, d = np.concatenate([z, zm, -zm * F(16)]), np.concatenate([d, dm, dm * F(4)])
    y0 = (F(1) / d).astype(F)
    if ulp:
        y0 = np.nextafter(y0, F(ulp) * F(np.inf))
    sl, sl2, ds = silu(z, d, y0)
    s = F(1) / d
    assert _same(sl, z / d) and _same(sl2, z / d)
    want = s.astype(np.float64) * (1 + z.astype(np.float64) * (F(1) - s).astype(np.float64))
    assert np.max(np.abs(ds - want)[:n]) <= 2.0**-23   # (z and d of a unit)


def test_saturated_units_and_special_values(silu):
    with np.errstate(all="ignore"):
        z = np.concatenate([np.linspace(-140, 140, 2801), -np.logspace(2, 38, 400), np.logspace(2, 38, 400),
                            [np.inf, -np.inf, np.nan, 0.0, -0.0]]).astype(F)
        d = (F(1) + np.exp(-z)).astype(F)
        y0 = (F(1) / d).astype(F)
        y0[np.abs(y0) < F(2.0**-126)] = 0   # a denormal estimate is returned as zero
        sl, sl2, ds = silu(z, d, y0)
        want, s = z / d, F(1) / d
        want_ds = s * (F(1) + z * (F(1) - s))
    edge = (d > F(2.0**126)) & np.isfinite(d)
    assert _same(sl[~edge], want[~edge]) and _same(sl2[~edge], want[~edge])
    assert np.all(np.abs(sl[edge] - want[edge]) <= 2e-36) and np.all(np.abs(sl2[edge] - want[edge]) <= 2e-36)
    assert np.array_equal(np.isnan(ds), np.isnan(want_ds))
    ok = ~np.isnan(ds)
    assert np.all(np.abs(ds[ok] - want_ds[ok]) <= 2.0**-22 * np.maximum(1, np.abs(want_ds[ok])))
