// Adjoint of the P2P short-range force (not in the paper; derived from the
// pair sum of Sec. 2, Eq. (tr)).
//
// For the loss L = sum_i w_i . a_i with a_i = G sum_l m_l g(r) d_il,
// d = x_l + s L - x_i, g = T / r^3, and h = g'(r) / r =
// -(3 T + (4 / sqrt(pi)) x^3 exp(-x^2)) / r^5 (x = r / 2 r_s), the gradient
// gathered over particle k's own neighbours (the P2P lists are symmetric) is
//   dL/dx_k = G [ m_k sum_l (g w_l + h (d.w_l) d) - sum_l m_l (g w_k + h (d.w_k) d) ]
//   dL/dm_k = -G sum_l g (w_l . d),                            d = d_kl,
// the delta function of the hard cutoff being left out.  Same wavefront
// mapping and work queue as the forward P2P kernel; the source records are
// (x, m) and (w, 0), both read with wave-uniform addresses.  g and h are
// evaluated exactly (float64: from the F table of f_table.h for r_cut <=
// 6 r_s, else truncation_T_f64; float32: erfcf and expf), or, in the float32
// r^2 form, read from quadratic tables in r^2.  Measured on 64^3 clustered
// particles, float32 r^2 tables: 932 us with one scalar load and wait per
// source and separate position terms, 618 us now (VALU and LDS issue); 48^3
// float64: 1350 us with the polynomial, 850 us from the F table (VALU).
#include "device.h"

#include <type_traits>

namespace pmfmm {
namespace {

constexpr double kFourOverSqrtPi = 2.25675833419102514780;
constexpr float kTwoOverSqrtPiF = 1.12837916709551257390f;
constexpr float kFourOverSqrtPiF = 2.25675833419102514780f;

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// The sums of one pair, from its g and h: with one common mass (EQ: source
// and target leaf have the same mass m everywhere, the rule in equal-mass
// sets) the two position terms combine to m [g u + h (d.u) d], u = w_l - w_k,
// added to A alone; otherwise A (times m_k at the end) and B take them apart.
// Not called for d = 0, the particle itself included: g = h = 0 would still
// make 0 times its own cotangent NaN where that is not finite.
template <bool EQ, class R, class V>
__device__ __forceinline__ void adj_sums(const V& q, const V& wl, const V& wk, R dx, R dy, R dz, R g,
                                         R h, R* A, R* Bv, R& gm) {
    const R dwl = fma(dz, wl.z, fma(dy, wl.y, dx * wl.x));
    if constexpr (EQ) {
        const R ux = wl.x - wk.x, uy = wl.y - wk.y, uz = wl.z - wk.z;
        const R hu = h * fma(dz, uz, fma(dy, uy, dx * ux));
        A[0] = fma(hu, dx, fma(g, ux, A[0]));
        A[1] = fma(hu, dy, fma(g, uy, A[1]));
        A[2] = fma(hu, dz, fma(g, uz, A[2]));
    } else {
        const R dwk = fma(dz, wk.z, fma(dy, wk.y, dx * wk.x));
        const R hl = h * dwl, gl = q.w * g, hk = q.w * h * dwk;
        A[0] = fma(hl, dx, fma(g, wl.x, A[0]));
        A[1] = fma(hl, dy, fma(g, wl.y, A[1]));
        A[2] = fma(hl, dz, fma(g, wl.z, A[2]));
        Bv[0] = fma(hk, dx, fma(gl, wk.x, Bv[0]));
        Bv[1] = fma(hk, dy, fma(gl, wk.y, Bv[1]));
        Bv[2] = fma(hk, dz, fma(gl, wk.z, Bv[2]));
    }
    gm = fma(-g, dwl, gm);
}

// Float64, polynomial T (cutoffs beyond 6 r_s).
template <bool EQ, bool SHIFTED>
__device__ __forceinline__ void adj_pair_f64(const double4& q, const double4& wl, double xk,
                                             double yk, double zk, const double4& wk, double sx,
                                             double sy, double sz, double rc2, double alpha,
                                             double* A, double* Bv, double& gm) {
    double dx, dy, dz, r2;
    {
#pragma clang fp contract(off)
        dx = q.x - xk;
        dy = q.y - yk;
        dz = q.z - zk;
        if (SHIFTED) {
            dx = dx + sx;
            dy = dy + sy;
            dz = dz + sz;
        }
        r2 = (dx * dx + dy * dy) + dz * dz;
    }
    if ((r2 > 0.0) & (r2 < rc2)) {
        const double idr = rsqrt(r2);
        const double x = r2 * idr * alpha;
        double ex;
        const double T = truncation_T_f64(x, &ex);
        const double idr2 = idr * idr;
        const double g = T * idr * idr2;
        const double h = -(3.0 * T + kFourOverSqrtPi * x * x * x * ex) * idr2 * idr2 * idr;
        adj_sums<EQ, double, double4>(q, wl, wk, dx, dy, dz, g, h, A, Bv, gm);
    }
}

// g and h of r^2 = s in the scaled units, from erfcf / expf.
__device__ __forceinline__ void adj_gh_f32(float s, float alpha, float& g, float& h) {
    const float idr = rsqrtf(s);
    const float x = s * idr * alpha;
    const float ex = expf(-x * x);
    const float T = erfcf(x) + kTwoOverSqrtPiF * x * ex;
    const float idr2 = idr * idr;
    g = T * idr * idr2;
    h = -(3.f * T + kFourOverSqrtPiF * x * x * x * ex) * idr2 * idr2 * idr;
}

// Float32, offsets in units of 1 / sigma (see BoxDev): g and h come out as
// sigma^-3 g and sigma^-5 h, d as sigma d, so A and B carry a factor
// sigma^-3 and gm sigma^-2, which the caller takes back out.
//
// TAB (the r^2 form; host builder in abi.cpp): g and h as quadratics in
// s = r'^2 on segments indexed by the float bits of s, in the units of the
// forward r^2 form (r_cut^2 = 2^kR2Emax), for s >= smin = 2^kAdjEmin (the floor
// keeps h's quadratic coefficient, which grows as s^(-9/2), a finite
// float).  A pair closer than that (r < 2^-18.5 r_cut, rare) takes g and h
// from erfcf / expf instead, at s no smaller than `tiny` = 2^kR2Emin, the
// forward's floor (float32 offsets resolve no closer pairs).  Coincident
// pairs (d = 0, the particle itself included) are left out.  Only lanes
// inside the cutoff read the six coefficients from LDS.
template <bool TAB, bool EQ>
__device__ __forceinline__ void adj_pair_f32(const float4 q, const float4 wl, float px, float py,
                                             float pz, const float4& wk, float rc2, float smin,
                                             uint32_t boff, float alpha, float tiny,
                                             const unsigned char* __restrict__ tab, float* A,
                                             float* Bv, float& gm) {
    const float dx = q.x - px, dy = q.y - py, dz = q.z - pz;
    // 0 < r2 < rc2 in one comparison: floats are ordered as their bits, negative
    // ones last.  TAB: 2^-126 less (nothing to any r2 that is not below 2^-102,
    // r < 2^-56 r_cut) makes a zero negative.  64^3 adjoint against two
    // comparisons: exact form 1478 -> 1445 us, tables 599 -> 589.
    const float r2 = fmaf(dz, dz, fmaf(dy, dy, TAB ? fmaf(dx, dx, -0x1p-126f) : dx * dx));
    const uint32_t least = TAB ? 0u : 1u;
    if (__float_as_uint(r2) - least < __float_as_uint(rc2) - least) {
        float g, h;
        if (TAB && r2 >= smin) {
            // (g c0, g c1), (h c0, h c1), (g c2, h c2) pairs of the row
            const unsigned char* c = tab + (((__float_as_uint(r2) >> (23 - kAdjBits)) << 3) + boff);
            const float2 g01 = *reinterpret_cast<const float2*>(c);
            const float2 h01 = *reinterpret_cast<const float2*>(c + 8 * kAdjPlane);
            const float2 c2 = *reinterpret_cast<const float2*>(c + 16 * kAdjPlane);
            g = fmaf(fmaf(c2.x, r2, g01.y), r2, g01.x);
            h = fmaf(fmaf(c2.y, r2, h01.y), r2, h01.x);
        } else {
            adj_gh_f32(TAB ? fmaxf(r2, tiny) : r2, alpha, g, h);
        }
        adj_sums<EQ, float, float4>(q, wl, wk, dx, dy, dz, g, h, A, Bv, gm);
    }
}

// Float64 from the F table (f_table.h): g = F / (2 r_s)^3 and h = 2 F' /
// (2 r_s)^5, where y F' = -(3/2) F - (2 / sqrt(pi)) exp(-y) gives h without
// another polynomial: every term has one sign, so nothing cancels.
// exp(-y) = exp(-(segment middle)) exp(-t), the first factor from the table,
// the second a Taylor polynomial (|t| <= y / 256 <= 0.036: the t^8 term left
// out is below 6e-17).  A, B and gm carry the factor (2 r_s)^3.
template <bool EQ, bool SHIFTED, bool END>
__device__ __forceinline__ void adj_pair_f64_F(const double4& q, const double4& wl, double xk,
                                               double yk, double zk, const double4& wk, double sx,
                                               double sy, double sz, const FTab<END>& T, double* A,
                                               double* Bv, double& gm) {
    double dx, dy, dz, r2;
    {
#pragma clang fp contract(off)
        dx = q.x - xk;
        dy = q.y - yk;
        dz = q.z - zk;
        if (SHIFTED) {
            dx = dx + sx;
            dy = dy + sy;
            dz = dz + sz;
        }
        r2 = (dx * dx + dy * dy) + dz * dz;
    }
    if ((r2 > 0.0) & (r2 < T.rc2)) {
        const double y = r2 * T.a2;
        const uint32_t hi = (uint32_t)__double2hiint(y);
        double g, e;
        if (hi >= (uint32_t)(1023 + kFEmin) << 20) {
            double t;
            const unsigned char* row;
            g = f_lookup(T, y, hi, &t, &row);
            double p = fma(t, -1.0 / 5040, 1.0 / 720);
            p = fma(t, p, -1.0 / 120);
            p = fma(t, p, 1.0 / 24);
            p = fma(t, p, -1.0 / 6);
            p = fma(t, p, 0.5);
            p = fma(t, p, -1.0);
            p = fma(t, p, 1.0);
            e = *reinterpret_cast<const double*>(row + 6 * kFPlane) * p;
        } else {
            g = f_close(y);
            e = 1.0 - y;
        }
        double iy = __builtin_amdgcn_rcp(y);   // 1 / y
        iy = fma(iy, fma(-y, iy, 1.0), iy);
        iy = fma(iy, fma(-y, iy, 1.0), iy);
        const double h = -T.a2 * iy * fma(kFourOverSqrtPi, e, 3.0 * g);
        adj_sums<EQ, double, double4>(q, wl, wk, dx, dy, dz, g, h, A, Bv, gm);
    }
}

template <class V, int N>
struct SrcN {
    V v[N];
};
__device__ __forceinline__ void pin4(const float4& a) {
    asm volatile("" ::"s"(a.x), "s"(a.y), "s"(a.z), "s"(a.w));
}
__device__ __forceinline__ void pin4(const double4& a) {
    asm volatile("" ::"s"(a.x), "s"(a.y), "s"(a.z), "s"(a.w));
}

// N sources of a j leaf and their cotangents by wave-uniform loads ahead of
// the pairs that need them: one load and wait per source took 0.3 of the
// float32 adjoint's time.  Reads past the leaf are never evaluated
// (kReadAhead).
template <int N, class V, class F>
__device__ __forceinline__ void adj_leaf(const V* __restrict__ src, const V* __restrict__ wsrc, int nj,
                                         uint64_t live, F pair) {
    for (int k = 0; k < nj; k += N) {
        const uint32_t g = (uint32_t)(live >> k) & ((1u << N) - 1u);
        if (g == 0) continue;
        const SrcN<V, N> b = *reinterpret_cast<const SrcN<V, N>*>(src + k);
        const SrcN<V, N> w = *reinterpret_cast<const SrcN<V, N>*>(wsrc + k);
#pragma unroll
        for (int u = 0; u < N; ++u) {
            pin4(b.v[u]);
            pin4(w.v[u]);
        }
#pragma unroll
        for (int u = 0; u < N; ++u)
            if (g & (1u << u)) pair(b.v[u], w.v[u]);
    }
}

enum AdjForm : int {
    kAdjF32 = 0,      // float32, erfcf / expf
    kAdjF32Tab = 1,   // float32, g and h tables in LDS (kAdjTableBytes)
    kAdjF64 = 2,      // float64, polynomial T
    kAdjF64Tab = 3,   // float64, F table in LDS (kFAdjTableBytes)
    kAdjF64End = 4    // the same, its last octave in use
};
constexpr bool adj_f_tab(int form) { return form == kAdjF64Tab || form == kAdjF64End; }
constexpr bool adj_f32(int form) { return form == kAdjF32 || form == kAdjF32Tab; }
constexpr int adj_lds(int form) {
    return form == kAdjF32Tab ? kAdjTableBytes : adj_f_tab(form) ? kFAdjTableBytes : 0;
}

// Waves per SIMD to leave room for.  Float32: eight (64 VGPRs, a few
// spills outside the pair loops; 64^3 adjoint 618 us against 662 us with the
// 77 VGPRs and six waves the compiler takes by itself).
constexpr int adj_min_waves(int form) { return adj_f32(form) ? 8 : form == kAdjF64 ? 3 : 1; }

template <int FORM>
__global__ void __launch_bounds__(FORM == kAdjF64 ? 256 : 1024, adj_min_waves(FORM))
adjoint_kernel(const double4* __restrict__ x64, const float4* __restrict__ x32,
               const double4* __restrict__ w64, const float4* __restrict__ w32,
               const int4* __restrict__ leaf, const double4* __restrict__ leafc,
               const int32_t* __restrict__ p2p_js, const int4* __restrict__ items,
               const int32_t* __restrict__ queue, int32_t n_items, int32_t* __restrict__ counter,
               double* __restrict__ partial, const BoxDev* __restrict__ boxes,
               const void* __restrict__ table) {
    extern __shared__ __align__(16) unsigned char adj_lds_mem[];
    if constexpr (adj_lds(FORM) != 0) {
        const uint4* src = reinterpret_cast<const uint4*>(table);
        uint4* dst = reinterpret_cast<uint4*>(adj_lds_mem);
        for (int i = threadIdx.x; i < adj_lds(FORM) / 16; i += blockDim.x) dst[i] = src[i];
        __syncthreads();
    }
    const int lane = threadIdx.x & 63;
    ItemCursor cur = item_cursor();
    for (;;) {
        const int q = take_item(cur, lane, n_items, counter);
        if (q < 0) break;
        const int slot = uni(queue[q]);
        const int4 it = items[slot];
        const int il = uni(it.x), t0 = uni(it.y), t1 = uni(it.z);
        const int4 li = leaf[il];
        const int ni = uni(li.y);
        const int pk = uni(li.x) + (lane < ni ? lane : 0);
        const BoxDev bx = boxes[uni(li.z)];
        const double4 ci = leafc[il];
        double A[3] = {0.0, 0.0, 0.0}, Bv[3] = {0.0, 0.0, 0.0}, gm = 0.0;
        const double mk = x64[pk].w;
        if constexpr (adj_f32(FORM)) {
            const float4 pv = x32[pk];
            const float4 wk = w32[pk];
            float3 lo = make_float3(pv.x, pv.y, pv.z), hi = lo;
            wave_box(lo, hi);
            // boff = -(row of 2^kAdjEmin) * 8 mod 2^32, kept opaque (an empty
            // asm on its scalar register) so that the address is one shift
            // and one shift-add and the three reads take their plane offsets
            // as immediates
            uint32_t boff = 0u - (((uint32_t)(127 + kAdjEmin) << kAdjBits) << 3);
            asm volatile("" : "+s"(boff));
            const float smin = __uint_as_float((uint32_t)(127 + kAdjEmin) << 23);
            const float rc2 = bx.rc2_f, alpha = bx.alpha_f, tiny = bx.tiny_f;
            for (int tb = t0; tb < t1; tb += 64) {
                const int nt = min(64, t1 - tb);
                const TaskLanes tl = load_tasks(p2p_js, tb + min(lane, nt - 1), leaf, leafc, ci, bx.L,
                                                bx.sigma);
                int jn = lane_of(tl.first, 0), nn = lane_of(tl.count, 0);
                float4 qn = x32[jn + min(lane, nn - 1)];
                for (int k = 0; k < nt; ++k) {
                    const float4 ql = qn;
                    const float4* __restrict__ src = x32 + jn;
                    const float4* __restrict__ wsrc = w32 + jn;
                    const int nj = nn;
                    if (k + 1 < nt) {
                        jn = lane_of(tl.first, k + 1);
                        nn = lane_of(tl.count, k + 1);
                        qn = x32[jn + min(lane, nn - 1)];
                    }
                    const float offx = lane_of(tl.ox, k), offy = lane_of(tl.oy, k),
                                offz = lane_of(tl.oz, k);
                    const bool eq = lane_of(tl.same, k) != 0;
                    const float px = pv.x - offx, py = pv.y - offy, pz = pv.z - offz;
                    float a[3] = {0.f, 0.f, 0.f}, b[3] = {0.f, 0.f, 0.f}, g = 0.f;
                    const uint64_t live =
                        live_f32(ql, nj, lane, make_float3(lo.x - offx, lo.y - offy, lo.z - offz),
                                 make_float3(hi.x - offx, hi.y - offy, hi.z - offz), rc2);
                    constexpr bool kTab = FORM == kAdjF32Tab;
                    if (eq)
                        adj_leaf<4>(src, wsrc, nj, live, [&](const float4& q, const float4& w) {
                            adj_pair_f32<kTab, true>(q, w, px, py, pz, wk, rc2, smin, boff, alpha,
                                                     tiny, adj_lds_mem, a, b, g);
                        });
                    else
                        adj_leaf<4>(src, wsrc, nj, live, [&](const float4& q, const float4& w) {
                            adj_pair_f32<kTab, false>(q, w, px, py, pz, wk, rc2, smin, boff, alpha,
                                                      tiny, adj_lds_mem, a, b, g);
                        });
                    for (int c = 0; c < 3; ++c) {
                        A[c] += (double)a[c];
                        Bv[c] += (double)b[c];
                    }
                    gm += (double)g;
                }
            }
            const double s2 = bx.sigma * bx.sigma, s3 = s2 * bx.sigma;
            for (int c = 0; c < 3; ++c) {
                A[c] *= s3;
                Bv[c] *= s3;
            }
            gm *= s2;
        } else {
            const double4 pv = x64[pk];
            const double4 wk = w64[pk];
            const FTab<FORM == kAdjF64End> T = f_tab<FORM == kAdjF64End>(adj_lds_mem, bx.rc2, bx.alpha);
            double3 lo = make_double3(pv.x, pv.y, pv.z), hi = lo;
            wave_box(lo, hi);
            for (int tb = t0; tb < t1; tb += 64) {
                const int nt = min(64, t1 - tb);
                const TaskLanes64 tl =
                    load_tasks64(p2p_js, tb + min(lane, nt - 1), leaf, leafc, ci.w);
                int jn = lane_of(tl.first, 0), cn = lane_of(tl.count_code, 0);
                double4 qn = x64[jn + min(lane, (cn >> 5) - 1)];
                for (int k = 0; k < nt; ++k) {
                    const double4 ql = qn;
                    const double4* __restrict__ src = x64 + jn;
                    const double4* __restrict__ wsrc = w64 + jn;
                    const int nj = cn >> 5, s = cn & 31;
                    if (k + 1 < nt) {
                        jn = lane_of(tl.first, k + 1);
                        cn = lane_of(tl.count_code, k + 1);
                        qn = x64[jn + min(lane, (cn >> 5) - 1)];
                    }
                    const bool eq = lane_of(tl.mass, k) == 2;
                    double sx, sy, sz;
                    image_shift(s, bx.L, sx, sy, sz);
                    const uint64_t live =
                        s == 13 ? live_f64<false>(ql, nj, lane, lo, hi, 0.0, 0.0, 0.0, bx.rc2)
                                : live_f64<true>(ql, nj, lane, lo, hi, sx, sy, sz, bx.rc2);
                    auto pairs = [&](auto eqc, auto shc) {
                        constexpr bool kEq = decltype(eqc)::value, kSh = decltype(shc)::value;
                        adj_leaf<adj_f_tab(FORM) ? 2 : 1>(src, wsrc, nj, live, [&](const double4& q, const double4& w) {
                            if constexpr (adj_f_tab(FORM))
                                adj_pair_f64_F<kEq, kSh>(q, w, pv.x, pv.y, pv.z, wk, sx, sy, sz, T, A,
                                                         Bv, gm);
                            else
                                adj_pair_f64<kEq, kSh>(q, w, pv.x, pv.y, pv.z, wk, sx, sy, sz, bx.rc2,
                                                       bx.alpha, A, Bv, gm);
                        });
                    };
                    if (s == 13) {
                        if (eq) pairs(std::true_type{}, std::false_type{});
                        else pairs(std::false_type{}, std::false_type{});
                    } else {
                        if (eq) pairs(std::true_type{}, std::true_type{});
                        else pairs(std::false_type{}, std::true_type{});
                    }
                }
            }
            if constexpr (adj_f_tab(FORM)) {
                const double a3 = T.a2 * bx.alpha;
                for (int c = 0; c < 3; ++c) {
                    A[c] *= a3;
                    Bv[c] *= a3;
                }
                gm *= a3;
            }
        }
        double* dst = partial + (size_t)slot * 256;
        dst[lane] = mk * A[0] - Bv[0];
        dst[64 + lane] = mk * A[1] - Bv[1];
        dst[128 + lane] = mk * A[2] - Bv[2];
        dst[192 + lane] = gm;
    }
}

__global__ void __launch_bounds__(256)
adj_reduce_kernel(const int4* __restrict__ leaf, const int32_t* __restrict__ leaf_slot,
                  const double* __restrict__ partial, const double4* __restrict__ far,
                  const int32_t* __restrict__ perm,
                  const BoxDev* __restrict__ boxes, double* __restrict__ gpos,
                  double* __restrict__ gmass, int32_t n_leaves) {
    const int l = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (l >= n_leaves) return;
    const int4 li = leaf[l];
    if (lane >= li.y) return;
    double g[4] = {0.0, 0.0, 0.0, 0.0};
    sum_slots(partial, leaf_slot[l], leaf_slot[l + 1], lane, g);
    if (far != nullptr) {
        const double4 f = far[li.x + lane];
        g[0] += f.x;
        g[1] += f.y;
        g[2] += f.z;
        g[3] += f.w;
    }
    const double G = boxes[li.z].G;
    const int o = perm[li.x + lane];
    gpos[3 * (size_t)o] = G * g[0];
    gpos[3 * (size_t)o + 1] = G * g[1];
    gpos[3 * (size_t)o + 2] = G * g[2];
    gmass[o] = G * g[3];
}

// w (caller order) -> leaf order, float64 and float32 records.
__global__ void gather_w_kernel(const double* __restrict__ w, const int32_t* __restrict__ perm,
                                double4* __restrict__ w64, float4* __restrict__ w32, int32_t n) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= n) return;
    const int o = perm[k];
    const double x = w[3 * (size_t)o], y = w[3 * (size_t)o + 1], z = w[3 * (size_t)o + 2];
    w64[k] = make_double4(x, y, z, 0.0);
    w32[k] = make_float4((float)x, (float)y, (float)z, 0.f);
}

template <int FORM>
int occ_adj(int wg_waves) {
    int blocks = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, adjoint_kernel<FORM>, 64 * wg_waves,
                                                     adj_lds(FORM)) != hipSuccess)
        return 1;
    return blocks > 0 ? blocks : 1;
}

}  // namespace

hipError_t launch_gather_w(const double* w, const int32_t* perm, double4* w64, float4* w32,
                           int32_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(gather_w_kernel, dim3((n + 255) / 256), dim3(256), 0, s, w, perm, w64, w32,
                       n);
    return hipGetLastError();
}

namespace {

template <int FORM>
hipError_t launch_form(const AdjArgs& a, int wg_waves, int grid_wgs, hipStream_t s) {
    hipLaunchKernelGGL(adjoint_kernel<FORM>, dim3(grid_wgs), dim3(64 * wg_waves), adj_lds(FORM), s,
                       a.x64, a.x32, a.w64, a.w32, a.leaf, a.leafc, a.p2p_js, a.items, a.queue,
                       a.n_items, a.counter, a.partial, a.boxes, a.table);
    return hipGetLastError();
}

int form_of(int mode, bool table) {
    if (is_fp32(mode)) return table ? kAdjF32Tab : kAdjF32;
    return table ? kAdjF64Tab : kAdjF64;
}

}  // namespace

hipError_t launch_adjoint(int mode, const AdjArgs& a, int wg_waves, int grid_wgs, hipStream_t s) {
    if (a.n_items == 0) return hipSuccess;
    switch (form_of(mode, a.table != nullptr)) {
        case kAdjF32: return launch_form<kAdjF32>(a, wg_waves, grid_wgs, s);
        case kAdjF32Tab: return launch_form<kAdjF32Tab>(a, wg_waves, grid_wgs, s);
        case kAdjF64: return launch_form<kAdjF64>(a, wg_waves, grid_wgs, s);
        default:
            if (a.f_end) return launch_form<kAdjF64End>(a, wg_waves, grid_wgs, s);
            return launch_form<kAdjF64Tab>(a, wg_waves, grid_wgs, s);
    }
}

hipError_t launch_adj_reduce(const AdjReduceArgs& a, hipStream_t s) {
    if (a.n_leaves == 0) return hipSuccess;
    hipLaunchKernelGGL(adj_reduce_kernel, dim3((a.n_leaves + 3) / 4), dim3(256), 0, s, a.leaf,
                       a.leaf_slot, a.partial, a.far, a.perm, a.boxes, a.grad_pos, a.grad_mass,
                       a.n_leaves);
    return hipGetLastError();
}

int adjoint_blocks_per_cu(int mode, int wg_waves, bool table) {
    switch (form_of(mode, table)) {
        case kAdjF32: return occ_adj<kAdjF32>(wg_waves);
        case kAdjF32Tab: return occ_adj<kAdjF32Tab>(wg_waves);
        case kAdjF64: return occ_adj<kAdjF64>(wg_waves);
        default: return occ_adj<kAdjF64Tab>(wg_waves);
    }
}

}  // namespace pmfmm
