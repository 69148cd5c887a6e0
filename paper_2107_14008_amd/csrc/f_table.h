// The segment table of the float64 exact pair form, built on the host.
//
// For cutoffs r_cut <= 6 r_s (x_c <= 3), with y = x^2 = (r / 2 r_s)^2,
// T(x) / r^3 = F(y) / (2 r_s)^3, F(y) = T(sqrt(y)) y^(-3/2), one function of y
// for every box.  F is tabulated on 2^kFBits segments per octave of y from
// 2^kFEmin to 9 (indexed by the high word of y), each a degree-6 polynomial in
// t = y - (segment middle) with c0 .. c3 in float64 and c4 .. c6 in float32 (44
// bytes a lookup; with c4 in float64 the LDS, which the lookups keep 75 % busy,
// took 7 % more time: 128^3 P2P 5.57 -> 6.00 ms).  What the roundings of c4 to c6
// change is taken up by c0 .. c3 up to its Chebyshev part of the same degree, an
// eighth of it for c4.  The kernels add the terms from t^4 on in float32 up to y
// = 8, where they are below 1e-8 of F (|t| <= y / 256), and with c4 widened to
// float64 when a cutoff lies beyond (up to 9e-8 of F; 2.3 % more time: 5.58 ->
// 5.70 ms).  So evaluated the table gives F within 2.6e-16 (relative; rms 7e-17)
// up to y = 4, 5.8e-16 (9e-17) up to 8, and 8e-16 (2.6e-16) in the last octave,
// where the terms past t^6 are up to 3.3e-16 of F.  The polynomial of
// truncation_T_f64 with its square roots and products stays within 2e-15.
// Pairs closer than y = 2^kFEmin take the series of F about y = 0.
//
// Layout: six arrays of kFRows eight-byte slots, (c4, c5), (c6, 0), (c0),
// (c1), (c2) and (c3), a multiple of 512 bytes apart, so that a lookup is an
// 8-byte, a 4-byte and two two-address LDS reads, all from one address
// register; a seventh holds exp(-(segment middle)) for the adjoint.
#pragma once

#include <cstddef>
#include <vector>

namespace pmfmm {

constexpr int kFBits = 7;
constexpr int kFEmin = -16;
constexpr int kFRows = 2496;
constexpr int kFPlane = kFRows * 8;
constexpr int kFTableBytes = 6 * kFPlane;
constexpr int kFAdjTableBytes = 7 * kFPlane;
constexpr int kFUsedRows = ((3 - kFEmin) << kFBits) + (1 << kFBits) / 8 + 1;   // y up to 9 and one more
constexpr double kFXcMax = 3.0;
constexpr double kFPlainMax = 7.999;   // largest y with the terms from t^4 on in float32
static_assert(kFUsedRows <= kFRows && kFPlane % 512 == 0, "rows of the F table");

// All kFAdjTableBytes of the table.
std::vector<unsigned char> build_f_table();

}  // namespace pmfmm
