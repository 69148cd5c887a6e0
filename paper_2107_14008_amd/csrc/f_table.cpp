#include "f_table.h"

#include <cmath>
#include <cstring>

namespace pmfmm {

// Per segment, with v = t / half width in [-1, 1]: the Taylor coefficients of F
// about the middle to order kN from the equation
//   y F' = -(3/2) F - (2 / sqrt(pi)) exp(-y)
// (one erfc and one exp per segment, in long double), cut to degree 6 by
// dropping the Chebyshev terms above it.
std::vector<unsigned char> build_f_table() {
    constexpr int kN = 14, kD = 6;
    using ld = long double;
    // cheb[k][j]: coefficient of v^j in T_k; low: v^m cut to degree kD
    ld cheb[kN + 1][kN + 1] = {}, low[kD + 1][kN + 1] = {};
    cheb[0][0] = 1;
    cheb[1][1] = 1;
    for (int k = 2; k <= kN; ++k)
        for (int j = 0; j <= kN; ++j)
            cheb[k][j] = (j > 0 ? 2 * cheb[k - 1][j - 1] : 0) - cheb[k - 2][j];
    for (int m = 0; m <= kN; ++m) {
        // v^m = 2^(1-m) sum_q C(m, q) T_(m-2q), the T_0 term halved
        ld binom = 1;
        for (int q = 0; 2 * q <= m; ++q) {
            const int k = m - 2 * q;
            const ld w = std::ldexp(binom, 1 - m) * (k == 0 ? 0.5L : 1.0L);
            if (k <= kD)
                for (int j = 0; j <= kD; ++j) low[j][m] += w * cheb[k][j];
            binom = binom * (m - q) / (q + 1);
        }
    }
    std::vector<unsigned char> out((size_t)kFAdjTableBytes, 0);
    const ld two_sqrt_pi = 1.128379167095512573896158903121545172L;
    for (int r = 0; r < kFUsedRows; ++r) {
        const int e = kFEmin + (r >> kFBits), j = r & ((1 << kFBits) - 1);
        const ld per = (ld)(1 << kFBits);
        const ld y = std::ldexp(1 + (j + 0.5L) / per, e), half = std::ldexp(0.5L / per, e);
        const ld x = std::sqrt(y), ey = std::exp(-y);
        ld f[kN + 1];
        f[0] = (std::erfc(x) + two_sqrt_pi * x * ey) / (y * x);
        // (n + 1) f_(n+1) y = -(n + 3/2) f_n - (2 / sqrt(pi)) (-1)^n exp(-y) / n!
        ld en = two_sqrt_pi * ey;
        for (int n = 0; n < kN; ++n) {
            f[n + 1] = -((n + 1.5L) * f[n] + en) / ((n + 1) * y);
            en = -en / (n + 1);
        }
        ld hp = 1;
        for (int n = 0; n <= kN; ++n) {
            f[n] *= hp;
            hp *= half;
        }
        // coefficients of v^k; those of v^4 to v^6 are rounded to float32 (of t^k),
        // highest first, and a rounding's v^k less T_k / 2^(k-1) goes into the
        // lower ones, so that only the T_k part of it is left
        ld c[kD + 1], width[kD + 1];
        width[0] = 1;
        for (int k = 0; k <= kD; ++k) {
            c[k] = 0;
            for (int n = 0; n <= kN; ++n) c[k] += low[k][n] * f[n];
            if (k > 0) width[k] = width[k - 1] * half;
        }
        for (int k = kD; k >= 4; --k) {
            const ld d = c[k] - (ld)(float)(c[k] / width[k]) * width[k];
            for (int j = 0; j < k; ++j) c[j] -= d * cheb[k][j] / std::ldexp(1.0L, k - 1);
            c[k] -= d;
        }
        unsigned char* slot = out.data() + (size_t)8 * r;
        for (int k = 0; k <= kD; ++k) {
            if (k < 4) {
                const double v = (double)(c[k] / width[k]);
                std::memcpy(slot + (size_t)(k + 2) * kFPlane, &v, 8);
            } else {
                const float v = (float)(c[k] / width[k]);
                std::memcpy(slot + (size_t)(k < 6 ? 0 : 1) * kFPlane + (k == 5 ? 4 : 0), &v, 4);
            }
        }
        const double em = (double)ey;
        std::memcpy(out.data() + (size_t)8 * r + (size_t)6 * kFPlane, &em, 8);
    }
    return out;
}

}  // namespace pmfmm
