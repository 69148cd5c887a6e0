"""The table of the float64 exact pair form (csrc/f_table.cpp): its rows, read
and evaluated as the kernels do, against 40-digit values of
F(y) = T(sqrt(y)) y^(-3/2), T(x) = erfc(x) + (2x / sqrt(pi)) exp(-x^2)."""

import ctypes
import os
import subprocess

import mpmath as mp
import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2107_14008_amd", "csrc")

# the steps of f_lookup (device.h)
SHIM = r"""
#include "f_table.h"
#include <cmath>
#include <cstdint>
#include <cstring>
using namespace pmfmm;
static double f64(const unsigned char* p) { double v; std::memcpy(&v, p, 8); return v; }
static float f32(const unsigned char* p) { float v; std::memcpy(&v, p, 4); return v; }
extern "C" void lookup(const double* y, double* F, double* em, double* mid, long n, int end) {
    const auto table = build_f_table();
    for (long i = 0; i < n; ++i) {
        uint64_t b;
        std::memcpy(&b, &y[i], 8);
        const uint32_t hi = (uint32_t)(b >> 32), sh = 20 - kFBits;
        const unsigned char* c = table.data() + 8 * ((size_t)(hi >> sh) - ((size_t)(1023 + kFEmin) << kFBits));
        const uint64_t mb = (uint64_t)((hi >> sh << sh) | (1u << (sh - 1))) << 32;
        std::memcpy(&mid[i], &mb, 8);
        const double t = y[i] - mid[i];
        const float p = std::fmaf(f32(c + kFPlane), (float)t, f32(c + 4));
        double f = end ? std::fma((double)p, t, (double)f32(c)) : (double)std::fmaf(p, (float)t, f32(c));
        for (int k : {5, 4, 3, 2}) f = std::fma(f, t, f64(c + (size_t)k * kFPlane));
        F[i] = f;
        em[i] = f64(c + (size_t)6 * kFPlane);
    }
}
"""


@pytest.fixture(scope="module")
def lookup(tmp_path_factory):
    d = tmp_path_factory.mktemp("ftable")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-shared", "-fPIC", f"-I{CSRC}",
                    str(d / "shim.cpp"), os.path.join(CSRC, "f_table.cpp"), "-o", str(d / "f.so")],
                   check=True)
    fn = ctypes.CDLL(str(d / "f.so")).lookup

    def run(y, end):
        out = [np.empty(len(y)) for _ in range(3)]
        ptr = [ctypes.c_void_p(a.ctypes.data) for a in (y, *out)]
        fn(*ptr, ctypes.c_long(len(y)), ctypes.c_int(end))
        return out
    return run


# Bounds: half an ulp of the last step and half an ulp of c0 (2^-53 each,
# together 2.2e-16 of F); the steps before, scaled by |t F' / F| of at most
# (1.5 + y) / 256 (1e-17); the terms that degree 6 leaves out, 2 (h / 2)^7
# |F^(7)| / 7! / F for half width h: below 2e-17 to y = 8, 3.3e-16 in the octave
# from 8 on (h = 1 / 32); and the float32 rounding (2^-24) of the t^4 term,
# h^4 |F^(4)| / 4! / F, of c4 by an eighth and, unless c4 is widened (`end`), of
# the sum: 3e-17 to y = 4, 4.5e-16 to y = 8 (h = 1 / 64); an eighth 4e-16 beyond.
@pytest.mark.parametrize("lo,hi,end,tol", [(2.0 ** -16, 1.0, 0, 2.9e-16), (1.0, 4.0, 0, 2.9e-16),
                                           (4.0, 5.0625, 0, 7e-16), (5.0625, 7.999, 0, 7e-16),
                                           (2.0 ** -16, 4.0, 1, 2.9e-16), (4.0, 8.0, 1, 2.9e-16),
                                           (8.0, 9.0, 1, 9.5e-16)])
def test_rows_against_forty_digits(lookup, lo, hi, end, tol):
    mp.mp.dps = 40
    rng = np.random.default_rng(3)
    n = 6000
    y = np.exp(rng.uniform(np.log(lo), np.log(hi), n))
    # the ends of segments, where |t| is largest, and 8.375, near the largest
    # error a row had with c4 in float32
    seg = np.unique(np.ldexp(np.floor(np.ldexp(np.frexp(y)[0], 8)), np.frexp(y)[1] - 8))
    y = np.concatenate([y, seg[:500], np.nextafter(seg[:500], 0), [8.374953]])
    y = y[(y >= lo) & (y < hi)]
    F, em, mid = lookup(np.ascontiguousarray(y), end)
    worst = 0.0
    for k in range(len(y)):
        x = mp.sqrt(mp.mpf(float(y[k])))
        ref = (mp.erfc(x) + 2 * x / mp.sqrt(mp.pi) * mp.exp(-x * x)) / x ** 3
        worst = max(worst, float(abs(mp.mpf(float(F[k])) / ref - 1)))
        assert abs(em[k] / float(mp.exp(-mp.mpf(float(mid[k])))) - 1) <= 2.3e-16
    assert worst <= tol, worst
