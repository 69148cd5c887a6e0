// Long-range part of the force split (Sec. 2) on a periodic mesh: cloud in
// cell assignment, a 3D real FFT, the Gaussian-filtered Newtonian Green's
// function, the spectral gradient, three inverse FFTs in one batch and cloud in
// cell interpolation, in float64.
//
//   rho(g)  = (N / L)^3 sum_i m_i W(x_i - g L / N)        (CIC weights W)
//   phi(k)  = -4 pi G rho(k) exp(-k^2 r_s^2) / k^2 / C(k)^2,  phi(0) = 0,
//             C(k) = prod_a sinc^2(k_a L / 2N) (undoes the assignment and
//             the interpolation once each)
//   a_a(k)  = -i k_a phi(k), the Nyquist component of k_a set to zero
//   a(x_i)  = sum_g W(x_i - g L / N) a(g)
//
// exp(-k^2 r_s^2) is the transform of erf(r / 2 r_s) / r over that of 1 / r,
// so this force plus the short-range pair force of Eq. (tr) is Newton's.
// The FFTs are rocFFT's (through hipFFT), plain library transforms; the
// deposit uses float64 atomics, so sums agree run to run only to rounding.
#include "pm.h"

#include <cmath>
#include <new>

namespace pmfmm {
namespace {

constexpr double kPi = 3.14159265358979323846;

__device__ __forceinline__ double wrap_pm(double x, double L) {
#pragma clang fp contract(off)
    if (x >= 0.0 && x < L) return x;
    double y = x - L * floor(x / L);
    if (y >= L) y -= L;
    if (y < 0.0) y += L;
    if (!(y >= 0.0 && y < L)) y = 0.0;
    return y;
}

// Lower node and the two CIC weights along one axis.
__device__ __forceinline__ void cic_axis(double x, double L, int n, int& g, double& w0, double& w1) {
    const double u = wrap_pm(x, L) * ((double)n / L);
    const double fl = floor(u);
    const double f = u - fl;
    g = (int)fl;
    if (g >= n) g -= n;
    w0 = 1.0 - f;
    w1 = f;
}

__global__ void pm_zero(double* __restrict__ p, int64_t m) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < m) p[i] = 0.0;
}

__global__ void pm_deposit(const double* __restrict__ pos, const double* __restrict__ mass, int64_t np,
                           double L, int n, double* __restrict__ rho) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= np) return;
    int g[3];
    double w[3][2];
    for (int a = 0; a < 3; ++a) cic_axis(pos[3 * i + a], L, n, g[a], w[a][0], w[a][1]);
    const double inv_cell = (double)n / L;
    const double mi = mass[i] * inv_cell * inv_cell * inv_cell;
    for (int dx = 0; dx < 2; ++dx) {
        const int x = g[0] + dx < n ? g[0] + dx : 0;
        for (int dy = 0; dy < 2; ++dy) {
            const int y = g[1] + dy < n ? g[1] + dy : 0;
            for (int dz = 0; dz < 2; ++dz) {
                const int z = g[2] + dz < n ? g[2] + dz : 0;
                atomicAdd(&rho[((int64_t)x * n + y) * n + z], mi * w[0][dx] * w[1][dy] * w[2][dz]);
            }
        }
    }
}

// ---- Deposit by blocks of the mesh (pm_deposit above is the direct form)
//
// Eight float64 atomics per particle on a mesh shared by eight XCDs ran at
// 37 G/s whatever the particles' order: 451 us of the 690 us call at 2.1 M
// particles on 128^3.  Instead the particles are binned by block of the mesh
// (one counting sort into at most kPmBins bins), each workgroup sums one
// block's particles into an LDS tile (LDS atomics), writes the tile out
// plainly, and each node adds the tiles that hold it.  A block with more than
// kPmChunk particles is cut into several workgroups and tiles.
constexpr int kPmBins = 4096;
constexpr int kPmPer = 4096;      // particles of one workgroup of the sort
constexpr int kPmChunk = 4096;    // particles of one workgroup of the deposit

// Blocks of e[0] x e[1] x e[2] cells (the last ones of an axis may be
// smaller), nb[a] per axis; a tile holds (e[0] + 1)(e[1] + 1)(e[2] + 1) nodes.
struct PmBlocks {
    int n, e[3], sh[3], nb[3], tile;   // e[a] = 1 << sh[a]
    __host__ __device__ int count() const { return nb[0] * nb[1] * nb[2]; }
};

__device__ __forceinline__ int pm_bin(const PmBlocks& b, int gx, int gy, int gz) {
    return ((gx >> b.sh[0]) * b.nb[1] + (gy >> b.sh[1])) * b.nb[2] + (gz >> b.sh[2]);
}

// The particles of one workgroup of the sort, kPmEach per thread: all their
// positions are loaded before the first is binned (16 waves per workgroup;
// with 4 waves and one load in flight the two passes took 84 us at 2.1 M
// particles, now 67 us: 20 to count, 47 to scatter the 36-byte records).
constexpr int kPmThreads = 1024;
constexpr int kPmEach = kPmPer / kPmThreads;

struct PmSlice {
    double x[kPmEach][3];
    int bin[kPmEach];    // -1 past the end
};

__device__ __forceinline__ PmSlice pm_slice(const PmBlocks& b, const double* __restrict__ pos,
                                            int64_t np, double L) {
    PmSlice s;
    const int64_t i0 = (int64_t)blockIdx.x * kPmPer + threadIdx.x;
#pragma unroll
    for (int r = 0; r < kPmEach; ++r) {
        const int64_t i = i0 + r * kPmThreads;
        for (int a = 0; a < 3; ++a) s.x[r][a] = i < np ? pos[3 * i + a] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < kPmEach; ++r) {
        int g[3];
        double w0, w1;
        for (int a = 0; a < 3; ++a) cic_axis(s.x[r][a], L, b.n, g[a], w0, w1);
        s.bin[r] = i0 + r * kPmThreads < np ? pm_bin(b, g[0], g[1], g[2]) : -1;
    }
    return s;
}

// Particles per bin; base[wg bins + bin]: the workgroup's first slot in the
// bin (written for the bins it has particles of).
__global__ void __launch_bounds__(kPmThreads)
pm_bin_count(const double* __restrict__ pos, int64_t np, double L, PmBlocks b,
             uint32_t* __restrict__ count, uint32_t* __restrict__ base) {
    __shared__ uint32_t h[kPmBins];
    const int bins = b.count();
    const PmSlice s = pm_slice(b, pos, np, L);
    for (int k = threadIdx.x; k < bins; k += kPmThreads) h[k] = 0u;
    __syncthreads();
    for (int r = 0; r < kPmEach; ++r)
        if (s.bin[r] >= 0) atomicAdd(&h[s.bin[r]], 1u);
    __syncthreads();
    for (int k = threadIdx.x; k < bins; k += kPmThreads)
        if (h[k]) base[(size_t)blockIdx.x * bins + k] = atomicAdd(&count[k], h[k]);
}

// start[k]: first sorted particle of bin k; cstart[k]: first deposit chunk of
// bin k (both with a total at [bins]); clears count for the next launch.  One
// workgroup, four bins per thread.
__global__ void __launch_bounds__(1024)
pm_bin_scan(int bins, uint32_t* __restrict__ count, uint32_t* __restrict__ start,
            uint32_t* __restrict__ cstart) {
    __shared__ uint64_t part[1024];
    const int t = threadIdx.x;
    uint64_t v[kPmBins / 1024], sum = 0;
    for (int j = 0; j < kPmBins / 1024; ++j) {
        const int k = t * (kPmBins / 1024) + j;
        const uint32_t c = k < bins ? count[k] : 0u;
        v[j] = (uint64_t)c | ((uint64_t)((c + kPmChunk - 1) / kPmChunk) << 32);
        sum += v[j];
        if (k < bins) count[k] = 0u;
    }
    part[t] = sum;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        const uint64_t x = t >= off ? part[t - off] : 0ull;
        __syncthreads();
        part[t] += x;
        __syncthreads();
    }
    uint64_t run = part[t] - sum;
    for (int j = 0; j < kPmBins / 1024; ++j) {
        const int k = t * (kPmBins / 1024) + j;
        if (k <= bins) {
            start[k] = (uint32_t)run;
            cstart[k] = (uint32_t)(run >> 32);
        }
        run += v[j];
        if (k + 1 == kPmBins && bins == kPmBins) {
            start[bins] = (uint32_t)run;
            cstart[bins] = (uint32_t)(run >> 32);
        }
    }
}

// Particle records (x, y, z, m) and caller indices in bin order.
__global__ void __launch_bounds__(kPmThreads)
pm_bin_scatter(const double* __restrict__ pos, const double* __restrict__ mass, int64_t np, double L,
               PmBlocks b, const uint32_t* __restrict__ start, const uint32_t* __restrict__ base,
               double4* __restrict__ rec, uint32_t* __restrict__ idx) {
    __shared__ uint32_t off[kPmBins];
    const int bins = b.count();
    const PmSlice s = pm_slice(b, pos, np, L);
    for (int k = threadIdx.x; k < bins; k += kPmThreads)
        off[k] = start[k] + base[(size_t)blockIdx.x * bins + k];   // unused bins: any value
    __syncthreads();
    const int64_t i0 = (int64_t)blockIdx.x * kPmPer + threadIdx.x;
    for (int r = 0; r < kPmEach; ++r) {
        if (s.bin[r] < 0) continue;
        const int64_t i = i0 + r * kPmThreads;
        const uint32_t at = atomicAdd(&off[s.bin[r]], 1u);
        rec[at] = make_double4(s.x[r][0], s.x[r][1], s.x[r][2], mass[i]);
        idx[at] = (uint32_t)i;
    }
}

// The block and the particles [p0, p1) of deposit chunk c; false past the last.
struct PmChunk {
    int o[3];
    uint32_t p0, p1;
};

__device__ __forceinline__ bool pm_chunk(const PmBlocks& b, uint32_t c, const uint32_t* __restrict__ start,
                                         const uint32_t* __restrict__ cstart, PmChunk& k) {
    const int bins = b.count();
    if (c >= cstart[bins]) return false;
    int lo = 0, hi = bins - 1;   // the bin whose chunks hold c
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (cstart[mid] <= c) lo = mid; else hi = mid - 1;
    }
    k.o[0] = lo / (b.nb[2] * b.nb[1]) << b.sh[0];
    k.o[1] = lo / b.nb[2] % b.nb[1] << b.sh[1];
    k.o[2] = lo % b.nb[2] << b.sh[2];
    k.p0 = start[lo] + (c - cstart[lo]) * kPmChunk;
    k.p1 = min(start[lo + 1], k.p0 + kPmChunk);
    return true;
}

// One chunk of a block's particles into its tile.  Bound by the LDS's float64
// atomics: eight per particle.
constexpr int kPmTileThreads = 512;

__global__ void __launch_bounds__(kPmTileThreads)
pm_tile_deposit(const double4* __restrict__ rec, double L, PmBlocks b,
                const uint32_t* __restrict__ start, const uint32_t* __restrict__ cstart,
                double* __restrict__ tiles) {
    extern __shared__ double tile[];
    PmChunk k;
    if (!pm_chunk(b, blockIdx.x, start, cstart, k)) return;
    for (int q = threadIdx.x; q < b.tile; q += kPmTileThreads) tile[q] = 0.0;
    __syncthreads();
    const double inv_cell = (double)b.n / L;
    const int sy = b.e[2] + 1, sx = (b.e[1] + 1) * sy;
    for (uint32_t p = k.p0 + threadIdx.x; p < k.p1; p += kPmTileThreads) {
        const double4 q = rec[p];
        int gx, gy, gz;
        double wx[2], wy[2], wz[2];
        cic_axis(q.x, L, b.n, gx, wx[0], wx[1]);
        cic_axis(q.y, L, b.n, gy, wy[0], wy[1]);
        cic_axis(q.z, L, b.n, gz, wz[0], wz[1]);
        const double mi = q.w * inv_cell * inv_cell * inv_cell;
        double* t0 = tile + (gx - k.o[0]) * sx + (gy - k.o[1]) * sy + (gz - k.o[2]);
        for (int dx = 0; dx < 2; ++dx)
            for (int dy = 0; dy < 2; ++dy)
                for (int dz = 0; dz < 2; ++dz)
                    atomicAdd(t0 + dx * sx + dy * sy + dz, mi * wx[dx] * wy[dy] * wz[dz]);
    }
    __syncthreads();
    double* out = tiles + (size_t)blockIdx.x * b.tile;
    for (int q = threadIdx.x; q < b.tile; q += kPmTileThreads) out[q] = tile[q];
}

// One chunk of a block's particles from tiles of the three fields in LDS,
// written to the callers' places.  Bound by those scattered writes: 71 us at
// 2.1 M particles in any order; reading the fields directly in the caller's
// order takes 66 us where that order is the mesh's, and about 410 us in a
// random order.
__global__ void __launch_bounds__(kPmTileThreads)
pm_tile_interp(const double4* __restrict__ rec, const uint32_t* __restrict__ idx, double L, PmBlocks b,
               const uint32_t* __restrict__ start, const uint32_t* __restrict__ cstart,
               const double* __restrict__ fx, const double* __restrict__ fy,
               const double* __restrict__ fz, double* __restrict__ acc) {
    extern __shared__ double tile[];
    PmChunk k;
    if (!pm_chunk(b, blockIdx.x, start, cstart, k)) return;
    const int n = b.n, sy = b.e[2] + 1, sx = (b.e[1] + 1) * sy;
    const double* __restrict__ f[3] = {fx, fy, fz};
    for (int q = threadIdx.x; q < b.tile; q += kPmTileThreads) {
        const int lx = q / sx, ly = (q - lx * sx) / sy, lz = q - lx * sx - ly * sy;
        // (a smaller last block's tile repeats nodes past its own upper face)
        int x = k.o[0] + lx, y = k.o[1] + ly, z = k.o[2] + lz;
        x -= x >= n ? n : 0;
        y -= y >= n ? n : 0;
        z -= z >= n ? n : 0;
        if (x < n && y < n && z < n) {
            const int64_t node = ((int64_t)x * n + y) * n + z;
            for (int a = 0; a < 3; ++a) tile[a * b.tile + q] = f[a][node];
        }
    }
    __syncthreads();
    for (uint32_t p = k.p0 + threadIdx.x; p < k.p1; p += kPmTileThreads) {
        const double4 q = rec[p];
        const int64_t i = (int64_t)idx[p];
        int gx, gy, gz;
        double wx[2], wy[2], wz[2];
        cic_axis(q.x, L, n, gx, wx[0], wx[1]);
        cic_axis(q.y, L, n, gy, wy[0], wy[1]);
        cic_axis(q.z, L, n, gz, wz[0], wz[1]);
        const double* t0 = tile + (gx - k.o[0]) * sx + (gy - k.o[1]) * sy + (gz - k.o[2]);
        double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int dx = c >> 2, dy = (c >> 1) & 1, dz = c & 1;
            const double wt = wx[dx] * wy[dy] * wz[dz];
            const double* t = t0 + dx * sx + dy * sy + dz;
            s[0] += wt * t[0];
            s[1] += wt * t[b.tile];
            s[2] += wt * t[2 * b.tile];
        }
        acc[3 * i] = s[0];
        acc[3 * i + 1] = s[1];
        acc[3 * i + 2] = s[2];
    }
}

// rho of every node: its own block's tiles, and, on a block's lower face, the
// upper face of the blocks below (periodic).
// One workgroup per (x, y) line of nodes.
__global__ void __launch_bounds__(128)
pm_tile_sum(PmBlocks b, const uint32_t* __restrict__ cstart, const double* __restrict__ tiles,
            double* __restrict__ rho) {
    const int n = b.n;
    const int g[2] = {(int)blockIdx.y, (int)blockIdx.x};
    int blk[3][2], loc[3][2], m[3];
    auto place = [&](int a, int v) {
        blk[a][0] = v >> b.sh[a];
        loc[a][0] = v - (blk[a][0] << b.sh[a]);
        m[a] = 1;
        if (loc[a][0] == 0) {
            blk[a][1] = blk[a][0] == 0 ? b.nb[a] - 1 : blk[a][0] - 1;
            loc[a][1] = min(b.e[a], n - (blk[a][1] << b.sh[a]));
            m[a] = 2;
        }
    };
    place(0, g[0]);
    place(1, g[1]);
    for (int v = threadIdx.x; v < n; v += 128) {
        place(2, v);
        double s = 0.0;
        for (int x = 0; x < m[0]; ++x)
            for (int y = 0; y < m[1]; ++y)
                for (int z = 0; z < m[2]; ++z) {
                    const int k = (blk[0][x] * b.nb[1] + blk[1][y]) * b.nb[2] + blk[2][z];
                    const int at = (loc[0][x] * (b.e[1] + 1) + loc[1][y]) * (b.e[2] + 1) + loc[2][z];
                    const uint32_t c1 = cstart[k + 1];
                    for (uint32_t c = cstart[k]; c < c1; ++c) s += tiles[(size_t)c * b.tile + at];
                }
        rho[((int64_t)g[0] * n + g[1]) * n + v] = s;
    }
}

__device__ __forceinline__ double sinc(double x) { return x == 0.0 ? 1.0 : sin(x) / x; }

// One thread per mode of the half spectrum (n, n, n / 2 + 1): the three
// gradient spectra, scaled by 1 / n^3 for the unnormalised inverse FFT.
__global__ void pm_green(const double2* __restrict__ rk, int n, double L, double r_s, double G,
                         double2* __restrict__ ax, double2* __restrict__ ay, double2* __restrict__ az) {
    const int nzh = n / 2 + 1;
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)n * n * nzh;
    if (q >= total) return;
    const int iz = (int)(q % nzh);
    const int iy = (int)((q / nzh) % n);
    const int ix = (int)(q / ((int64_t)nzh * n));
    const double dk = 2.0 * kPi / L;
    // numpy fftfreq order: index n / 2 is -n / 2 (the Nyquist mode)
    const int mx = ix < (n + 1) / 2 ? ix : ix - n;
    const int my = iy < (n + 1) / 2 ? iy : iy - n;
    const int mz = iz < (n + 1) / 2 ? iz : iz - n;
    const double kx = dk * mx, ky = dk * my, kz = dk * mz;
    const double k2 = kx * kx + ky * ky + kz * kz;
    double2 zero = make_double2(0.0, 0.0);
    if (k2 == 0.0) {
        ax[q] = zero;
        ay[q] = zero;
        az[q] = zero;
        return;
    }
    const double h2 = 0.5 * L / (double)n;
    const double c = sinc(kx * h2) * sinc(ky * h2) * sinc(kz * h2);
    const double C = c * c;
    const double inv_n3 = 1.0 / ((double)n * (double)n * (double)n);
    const double gk = -4.0 * kPi * G * exp(-k2 * r_s * r_s) / k2 / (C * C) * inv_n3;
    const double2 r = rk[q];
    const double pr = r.x * gk, pi = r.y * gk;   // phi(k)
    const bool even = (n % 2) == 0;
    const double kxx = (even && ix == n / 2) ? 0.0 : kx;
    const double kyy = (even && iy == n / 2) ? 0.0 : ky;
    const double kzz = (even && iz == n / 2) ? 0.0 : kz;
    // -i k phi = (k pi, -k pr)
    ax[q] = make_double2(kxx * pi, -kxx * pr);
    ay[q] = make_double2(kyy * pi, -kyy * pr);
    az[q] = make_double2(kzz * pi, -kzz * pr);
}

__global__ void pm_interp(const double* __restrict__ pos, int64_t np, double L, int n,
                          const double* __restrict__ fx, const double* __restrict__ fy,
                          const double* __restrict__ fz, double* __restrict__ acc) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= np) return;
    int g[3];
    double w[3][2];
    for (int a = 0; a < 3; ++a) cic_axis(pos[3 * i + a], L, n, g[a], w[a][0], w[a][1]);
    double s[3] = {0.0, 0.0, 0.0};
    for (int dx = 0; dx < 2; ++dx) {
        const int x = g[0] + dx < n ? g[0] + dx : 0;
        for (int dy = 0; dy < 2; ++dy) {
            const int y = g[1] + dy < n ? g[1] + dy : 0;
            for (int dz = 0; dz < 2; ++dz) {
                const int z = g[2] + dz < n ? g[2] + dz : 0;
                const int64_t node = ((int64_t)x * n + y) * n + z;
                const double wt = w[0][dx] * w[1][dy] * w[2][dz];
                s[0] += wt * fx[node];
                s[1] += wt * fy[node];
                s[2] += wt * fz[node];
            }
        }
    }
    acc[3 * i] = s[0];
    acc[3 * i + 1] = s[1];
    acc[3 * i + 2] = s[2];
}

inline unsigned blocks_of(int64_t m) { return (unsigned)((m + 255) / 256); }

}  // namespace

namespace {

// Block edges for an n^3 mesh: at most kPmBins blocks, enough of them for the
// 256 CUs where the mesh allows it, tiles of 6 to 39 KB.
PmBlocks pm_blocks(int n) {
    PmBlocks b{};
    b.n = n;
    b.sh[0] = n <= 128 ? 3 : 4;
    b.sh[1] = b.sh[2] = n <= 64 ? 3 : 4;
    b.tile = 1;
    for (int a = 0; a < 3; ++a) {
        b.e[a] = 1 << b.sh[a];
        b.nb[a] = (n + b.e[a] - 1) / b.e[a];
        b.tile *= b.e[a] + 1;
    }
    return b;
}

// The block form's buffers for np particles; false when the direct form is to
// be used: meshes beyond 256^3 (more blocks than kPmBins), few particles (the
// whole call at 32^3 particles and mesh: 68 us by blocks, 100 us direct; the
// gain shrinks with the particles), far fewer particles than nodes (every
// node's tiles are moved twice: 100^3 particles on 256^3 nodes took 1497 us by
// blocks, 1457 direct), no memory, or buffers to grow while the stream is
// being captured.
constexpr int64_t kPmMinParticles = 16384;

// Room for one more retired buffer.
bool pm_may_retire(PMPlan& p) {
    try {
        p.retired.reserve(p.retired.size() + 1);
    } catch (const std::bad_alloc&) {
        return false;
    }
    return true;
}

bool pm_block_buffers(PMPlan& p, int64_t np, hipStream_t s) {
    if (p.n > 256 || np < kPmMinParticles || np > (int64_t)UINT32_MAX) return false;
    if (4 * np < (int64_t)p.n * p.n * p.n) return false;
    const PmBlocks b = pm_blocks(p.n);
    const size_t bins = (size_t)b.count(), wgs = (size_t)((np + kPmPer - 1) / kPmPer);
    const size_t chunks = bins + (size_t)(np / kPmChunk) + 1;
    const size_t words = 3 * (bins + 8) + wgs * bins;
    const size_t bytes[4] = {(size_t)np * 32, (size_t)np * 4, words * 4, chunks * b.tile * 8};
    bool fits = true;
    for (int k = 0; k < 4; ++k) fits = fits && p.blk_bytes[k] >= bytes[k];
    if (fits) return pm_may_retire(p);   // room to set the counts aside if a launch fails
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone) return false;
    for (int k = 0; k < 4; ++k) {
        if (p.blk_bytes[k] >= bytes[k]) continue;
        // half as much again, and the old buffer kept until pm_release: a
        // graph captured with it stays valid (all of them together take at
        // most twice the newest)
        const size_t want = p.blk[k] ? bytes[k] + bytes[k] / 2 : bytes[k];
        void* q = nullptr;
        if (!pm_may_retire(p)) return false;
        if (hipMalloc(&q, want) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        if (k == 2) {
            // here, where nothing is being captured and whatever comes of the
            // call: no later one has to know whether the counts are clear
            hipLaunchKernelGGL(pm_zero, dim3(blocks_of((int64_t)(bins + 1) / 2)), dim3(256), 0, s,
                               static_cast<double*>(q), (int64_t)((bins + 1) / 2));
            if (hipGetLastError() != hipSuccess) {
                (void)hipFree(q);
                return false;
            }
        }
        if (p.blk[k]) p.retired.push_back(p.blk[k]);
        p.blk[k] = q;
        p.blk_bytes[k] = want;
    }
    return pm_may_retire(p);
}

}  // namespace

hipError_t pm_plan(PMPlan& p, int n, hipStream_t s) {
    if (p.n == n && p.fwd != 0) {
        if (hipfftSetStream(p.fwd, s) != HIPFFT_SUCCESS || hipfftSetStream(p.inv, s) != HIPFFT_SUCCESS)
            return hipErrorUnknown;
        return hipSuccess;
    }
    pm_release(p);
    const int64_t n3 = (int64_t)n * n * n, nh = (int64_t)n * n * (n / 2 + 1);
    hipError_t e;
    if ((e = hipMalloc(&p.rho, n3 * sizeof(double))) != hipSuccess) return e;
    if ((e = hipMalloc(&p.rk, nh * 2 * sizeof(double))) != hipSuccess) return e;
    // the three spectra and the three fields, each set in one piece for the
    // batched inverse transform
    if ((e = hipMalloc(&p.gk[0], 3 * nh * 2 * sizeof(double))) != hipSuccess) return e;
    if ((e = hipMalloc(&p.field[0], 3 * n3 * sizeof(double))) != hipSuccess) return e;
    for (int a = 1; a < 3; ++a) {
        p.gk[a] = p.gk[0] + a * nh * 2;
        p.field[a] = p.field[0] + a * n3;
    }
    if (hipfftPlan3d(&p.fwd, n, n, n, HIPFFT_D2Z) != HIPFFT_SUCCESS) return hipErrorUnknown;
    // (the default layout, which is this one: spelt out, the library compiles
    // kernels of its own for it, 340 ms once per process and mesh size)
    int dims[3] = {n, n, n};
    if (hipfftPlanMany(&p.inv, 3, dims, nullptr, 1, 0, nullptr, 1, 0, HIPFFT_Z2D, 3) != HIPFFT_SUCCESS)
        return hipErrorUnknown;
    if (hipfftSetStream(p.fwd, s) != HIPFFT_SUCCESS || hipfftSetStream(p.inv, s) != HIPFFT_SUCCESS)
        return hipErrorUnknown;
    p.n = n;
    return hipSuccess;
}

void pm_release(PMPlan& p) {
    if (p.fwd) (void)hipfftDestroy(p.fwd);
    if (p.inv) (void)hipfftDestroy(p.inv);
    p.fwd = p.inv = 0;
    if (p.rho) (void)hipFree(p.rho);
    if (p.rk) (void)hipFree(p.rk);
    p.rho = nullptr;
    p.rk = nullptr;
    for (int k = 0; k < 4; ++k) {
        if (p.blk[k]) (void)hipFree(p.blk[k]);
        p.blk[k] = nullptr;
        p.blk_bytes[k] = 0;
    }
    for (void* q : p.retired) (void)hipFree(q);
    p.retired.clear();
    if (p.gk[0]) (void)hipFree(p.gk[0]);
    if (p.field[0]) (void)hipFree(p.field[0]);
    for (int a = 0; a < 3; ++a) {
        p.gk[a] = nullptr;
        p.field[a] = nullptr;
    }
    p.n = 0;
}

hipError_t pm_long_range(PMPlan& p, const double* pos, const double* mass, int64_t np, double L,
                         double r_s, double G, double* acc, hipStream_t s) {
    const int n = p.n;
    const int64_t n3 = (int64_t)n * n * n, nh = (int64_t)n * n * (n / 2 + 1);
    hipError_t e;
    const bool blocks = pm_block_buffers(p, np, s);
    double4* rec = static_cast<double4*>(p.blk[0]);
    uint32_t* idx = static_cast<uint32_t*>(p.blk[1]);
    if (blocks) {
        const PmBlocks b = pm_blocks(n);
        const int bins = b.count();
        uint32_t* count = static_cast<uint32_t*>(p.blk[2]);
        uint32_t* start = count + bins + 8;
        uint32_t* cstart = start + bins + 8;
        uint32_t* base = cstart + bins + 8;
        const unsigned wgs = (unsigned)((np + kPmPer - 1) / kPmPer);
        const unsigned chunks = (unsigned)(bins + np / kPmChunk + 1);
        hipLaunchKernelGGL(pm_bin_count, dim3(wgs), dim3(kPmThreads), 0, s, pos, np, L, b, count, base);
        hipLaunchKernelGGL(pm_bin_scan, dim3(1), dim3(1024), 0, s, bins, count, start, cstart);
        hipLaunchKernelGGL(pm_bin_scatter, dim3(wgs), dim3(kPmThreads), 0, s, pos, mass, np, L, b, start, base,
                           rec, idx);
        hipLaunchKernelGGL(pm_tile_deposit, dim3(chunks), dim3(kPmTileThreads), (size_t)b.tile * 8, s, rec, L, b,
                           start, cstart, static_cast<double*>(p.blk[3]));
        hipLaunchKernelGGL(pm_tile_sum, dim3(n, n), dim3(128), 0, s, b, cstart,
                           static_cast<const double*>(p.blk[3]), p.rho);
        if ((e = hipGetLastError()) != hipSuccess) {
            // the counts may have been added to and not cleared
            p.retired.push_back(p.blk[2]);
            p.blk[2] = nullptr;
            p.blk_bytes[2] = 0;
            return e;
        }
    } else {
        hipLaunchKernelGGL(pm_zero, dim3(blocks_of(n3)), dim3(256), 0, s, p.rho, n3);
        if (np > 0)
            hipLaunchKernelGGL(pm_deposit, dim3(blocks_of(np)), dim3(256), 0, s, pos, mass, np, L, n,
                               p.rho);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (hipfftExecD2Z(p.fwd, p.rho, reinterpret_cast<hipfftDoubleComplex*>(p.rk)) != HIPFFT_SUCCESS)
        return hipErrorUnknown;
    hipLaunchKernelGGL(pm_green, dim3(blocks_of(nh)), dim3(256), 0, s,
                       reinterpret_cast<const double2*>(p.rk), n, L, r_s, G,
                       reinterpret_cast<double2*>(p.gk[0]), reinterpret_cast<double2*>(p.gk[1]),
                       reinterpret_cast<double2*>(p.gk[2]));
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (hipfftExecZ2D(p.inv, reinterpret_cast<hipfftDoubleComplex*>(p.gk[0]), p.field[0]) != HIPFFT_SUCCESS)
        return hipErrorUnknown;
    if (blocks) {
        const PmBlocks b = pm_blocks(n);
        const uint32_t* start = static_cast<const uint32_t*>(p.blk[2]) + b.count() + 8;
        hipLaunchKernelGGL(pm_tile_interp, dim3((unsigned)(b.count() + np / kPmChunk + 1)),
                           dim3(kPmTileThreads), (size_t)b.tile * 24, s, rec, idx, L, b, start,
                           start + b.count() + 8, p.field[0], p.field[1], p.field[2], acc);
    } else if (np > 0) {
        hipLaunchKernelGGL(pm_interp, dim3(blocks_of(np)), dim3(256), 0, s, pos, np, L, n, p.field[0],
                           p.field[1], p.field[2], acc);
    }
    return hipGetLastError();
}

}  // namespace pmfmm
