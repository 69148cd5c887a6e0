// On-GPU planner: the ORB tree (Sec. 2), the dual walk into P2P and M2L
// task lists (Sec. 3) and the TaskGroup / GroupIdx CSR with its work items
// (Sec. 3.2), built from particles already in HBM.  Same readings as the
// host planner (plan.cpp), and the same results bit for bit: every geometry
// decision is the same rounded float64 operation in the same order.
//
// ORB without per-cell sorting: the particles are sorted once per axis by
// (coordinate, caller index) with a stable radix sort; the shape of the tree
// (which cell holds which range of positions) depends on the particle count
// alone and comes from the host.  Level by level, each splitting cell reads
// its bounds from the ends of its three sorted ranges, marks the floor(n/2)
// first particles of its split axis as "left", and every axis list is
// partitioned stably (prefix sums of the left marks), which keeps each child
// range sorted on every axis.  Once a subtree holds at most 8192 particles
// and 1024 cells, one workgroup finishes it in LDS (k_orb_fused), so the
// launches per level are paid only for the top levels.
//
// Dual walk: level-synchronous over a frontier of cell pairs (the canonical
// half of the symmetric walk); one thread per pair classifies it and appends
// P2P keys, M2L keys (each with its mirror) or child pairs with one atomic
// per counter and workgroup.  The keys (i, j << 5 | shift) are counted per
// row i and placed into CSR rows, and each row is sorted (k_row_*), which
// yields the canonical (i, j, shift) order.
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "gpu_plan.h"

namespace pmfmm {
namespace {

constexpr double kGuard = 0x1p-40;

struct WalkBox {
    double L, rc2_drop, rc2_m2l, th2;
    int32_t use_m2l, centre_cut;   // centre_cut: M2L by centre distance, else drop
    double rc2;
};

__device__ __forceinline__ double wrap_coord(double x, double L) {
#pragma clang fp contract(off)
    if (x >= 0.0 && x < L) return x;
    double y = x - L * floor(x / L);
    if (y >= L) y -= L;
    if (y < 0.0) y += L;
    if (!(y >= 0.0 && y < L)) y = 0.0;
    return y;
}

__device__ __forceinline__ int box_of(const int32_t* __restrict__ bf, int nbox, int i) {
    int lo = 0, hi = nbox - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (bf[mid] <= i) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// Order-preserving key of a non-negative double (+0 and -0 equal).
__device__ __forceinline__ uint64_t coord_key(double x) {
    return x == 0.0 ? 0ull : (uint64_t)__double_as_longlong(x);
}

// Sort key of a wrapped coordinate x in [0, L): floor(x 2^bits / L) with
// 24 or 32 bits, a non-decreasing function of x (a rounded product and a
// floor), so that sorting by it and then ordering each run of equal keys by
// x is the order by x.  24 bits (three 8-bit radix passes) up to
// kKey24Max particles, where a bin of L / 2^24 rarely holds two of them;
// beyond, the runs of equal keys would cost k_run_fix more than the fourth
// pass (measured at 256^3), and the key has 32 bits.
constexpr int64_t kKey24Max = int64_t(1) << 22;
__device__ __forceinline__ uint32_t coord_key(double x, double scale, double kmax) {
    const double t = x * scale;
    return t >= kmax ? (uint32_t)kmax : (uint32_t)t;
}

// The start of a build: the words of the planner's counters (wcount, with
// the walk's control words behind them) and the row counts to their initial
// values, in one launch.
constexpr int kCtlWords = 1024;         // walk control words, at wcount + kCtlAt
constexpr int kCtlAt = 32;
// wcount words: 0, 1 first bad position / mass (INT_MAX: none), 2 long-run flag
// of the coordinate sort, 4 .. 7 the host-driven walk's M2L depths, 8, 9
// candidate pairs, 10 items, 16, 17 smallest M2L depths (INT_MAX: none), 20 ..
// 23 the host-driven walk's counters

__global__ void k_init(int32_t* __restrict__ wcount, int32_t* __restrict__ rowcnt, int nrow,
                       int32_t* __restrict__ rowcnt_m2l, int nrow_m2l, int32_t* __restrict__ m2l_row,
                       int nm2l_row) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < kCtlAt + kCtlWords)
        wcount[i] = (i < 2 || i == 16 || i == 17) ? 0x7fffffff : 0;
    if (i < nrow) rowcnt[i] = 0;
    if (i < nrow_m2l) rowcnt_m2l[i] = 0;
    if (i < nm2l_row) m2l_row[i] = 0;
}

// Per particle: the input checks, the wrapped position and the three sort keys.
__global__ void k_prepare(const double* __restrict__ pos, const double* __restrict__ mass, int64_t n,
                          const int32_t* __restrict__ bf, int nbox,
                          const BoxDev* __restrict__ boxes, double* __restrict__ wpos,
                          uint32_t* __restrict__ keys, uint32_t* __restrict__ vals, int key_bits,
                          int* __restrict__ bad) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int b = box_of(bf, nbox, (int)i);
    const double L = boxes[b].L;
    const double range = key_bits == 24 ? 16777216.0 : 4294967296.0;
    const double scale = range / L;
    double x[3];
    for (int a = 0; a < 3; ++a) x[a] = pos[3 * i + a];
    const double m = mass[i];
    if (!(isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]))) atomicMin(&bad[0], (int)i);
    if (!(isfinite(m) && m >= 0.0)) atomicMin(&bad[1], (int)i);
    for (int a = 0; a < 3; ++a) {
        const double y = wrap_coord(x[a], L);
        wpos[3 * i + a] = y;
        keys[a * n + i] = coord_key(y, scale, range - 1.0);
        vals[a * n + i] = (uint32_t)i;
    }
}

// Full 64-bit keys of the wrapped coordinates (the fallback sort).
__global__ void k_keys64(const double* __restrict__ wpos, int64_t n, uint64_t* __restrict__ keys,
                         uint32_t* __restrict__ vals) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    for (int a = 0; a < 3; ++a) {
        keys[a * n + i] = coord_key(wpos[3 * i + a]);
        vals[a * n + i] = (uint32_t)i;
    }
}

// After the stable sort by the key, each run of equal keys of one axis
// list is in caller order; this puts it in coordinate order (stable, so
// equal coordinates stay in caller order).  The first position of a run of
// at most kRunMax elements sorts it in place (insertion sort).  A longer
// run is only checked: its start checks its first kRunMax - 1 neighbour
// pairs and every later position the pair it ends; any pair out of order
// sets *longrun, and the caller then sorts by the full 64-bit keys.
constexpr int kRunMax = 64;

__global__ void k_run_fix(const uint32_t* __restrict__ keys, uint32_t* __restrict__ vals, int64_t n,
                          const double* __restrict__ wpos, int* __restrict__ longrun) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= 3 * n) return;
    const int a = q >= n ? (q >= 2 * n ? 2 : 1) : 0;
    const int64_t s0 = (int64_t)a * n, s1 = s0 + n;
    const uint32_t h = keys[q];
    auto x_of = [&](int64_t p) { return wpos[3 * (size_t)vals[p] + a]; };
    if (q == s0 || keys[q - 1] != h) {
        if (q + 1 >= s1 || keys[q + 1] != h) return;   // a run of one
        if (q + kRunMax < s1 && keys[q + kRunMax] == h) {
            double prev = x_of(q);
            for (int64_t p = q + 1; p < q + kRunMax; ++p) {
                const double x = x_of(p);
                if (x < prev) {
                    atomicOr(longrun, 1);
                    return;
                }
                prev = x;
            }
            return;
        }
        int64_t e = q + 2;
        while (e < s1 && keys[e] == h) ++e;
        for (int64_t i = q + 1; i < e; ++i) {
            const uint32_t vi = vals[i];
            const double xi = wpos[3 * (size_t)vi + a];
            int64_t j = i - 1;
            while (j >= q) {
                const uint32_t vj = vals[j];
                if (!(xi < wpos[3 * (size_t)vj + a])) break;
                vals[j + 1] = vj;
                --j;
            }
            vals[j + 1] = vi;
        }
    } else if (q - kRunMax >= s0 && keys[q - kRunMax] == h) {
        // kRunMax or more positions into a long run (keys are sorted)
        if (x_of(q) < x_of(q - 1)) atomicOr(longrun, 1);
    }
}

__global__ void k_box_keys(const uint32_t* __restrict__ vals, int64_t n, const int32_t* __restrict__ bf,
                           int nbox, uint32_t* __restrict__ keys) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[i] = (uint32_t)box_of(bf, nbox, (int)vals[i]);
}

// One level of the level loop: the cells that split at this depth, in position
// order, and where each tile of kLvTile positions finds its first one.  Both
// depend on the shape of the tree alone and come from the host: a position's
// cell is then at most a step or two from its tile's first (the loop's cells
// hold more than kFuseM particles, or more than kFuseC cells), and no array of
// cells by position is read, partitioned and written at every level.
struct LevelCells {
    const int4* cells;      // (first position, count, cell id, left marks before it)
    const int32_t* tile;    // per tile: index of the first cell that ends beyond its start
    int count;
    int32_t* axis;          // per cell: split axis, written by k_level_flag
};

// The cell of position i, from index c on (c only grows); false if i is in no
// cell of the level.
__device__ __forceinline__ bool level_cell(const LevelCells& lv, int64_t i, int& c, int4& ci) {
    while (c < lv.count) {
        ci = lv.cells[c];
        if (i < (int64_t)ci.x + ci.y) return i >= ci.x;
        ++c;
    }
    return false;
}

// The stable partition of one level, with the left marks of the three lists
// (list a at [a n, (a + 1) n) of plist) computed where they are used instead
// of stored: a position's mark is its particle's left mark if its cell
// splits at this level, else 0.  A tile is the list positions [b T, (b + 1)
// T), T = 1024, of all three lists, whose cells are the same.  A splitting
// cell marks the first floor(count / 2) positions of its range in every list
// and nothing else is marked, so the marks before a cell's first position are
// the same in the three lists and known from the shape.  k_level_flag gives
// every particle its mark, k_level_sums looks the positions' marks up, keeps
// them as bits in list order and counts each tile's per list, and
// k_level_move counts them before every position (the tiles before its own,
// summed where they are needed, + the tile's words) and from the difference
// places the position.  The look-ups are random reads at a line per lane, so
// they are made once: with k_level_move looking them up again it took 189 us
// a level at 256^3 and 24 at 128^3, now 79 and 14.5 (read and write of the
// lists: 5.1 TB/s).
constexpr int kLvThreads = 256;
constexpr int kLvRounds = 4;
constexpr int kLvTile = kLvThreads * kLvRounds;   // 1024 positions of each list
constexpr int kLvWords = kLvTile / 64;            // mark words of each list's tile
static_assert(3 * kLvWords <= 64, "one wavefront scans the words");

// Per tile: the bounds of the cells it meets from the ends of their sorted
// ranges (six lanes of every wave, two dependent loads; one workgroup for the
// level's cells took a launch of its own), their split axes, and the left
// marks of its positions in the split axis's list, as bytes indexed by
// particle (a byte store needs no atomic).  A left mark is the value `gen`,
// another one at each level, so only the left half is written (scattered: 171
// us a level at 256^3 with both halves, now 112), but for the first level
// (`all`), which gives every particle of the loop's cells a value.  The tile
// that holds a cell's first position writes its bounds and axis.
__global__ void __launch_bounds__(kLvThreads)
k_level_flag(int64_t n, LevelCells lv, const uint32_t* __restrict__ plist,
             const double* __restrict__ wpos, double* __restrict__ clo, double* __restrict__ chi,
             uint8_t* __restrict__ flag, int gen, bool all) {
    const int64_t base = (int64_t)blockIdx.x * kLvTile, last = min(n, base + kLvTile);
    const int t = threadIdx.x, lane = t & 63;
    for (int c = lv.tile[blockIdx.x]; c < lv.count; ++c) {
        const int4 ci = lv.cells[c];
        if (ci.x >= last) break;
        const int a = min(lane >> 1, 2);
        const int64_t e = (lane & 1) ? (int64_t)ci.x + ci.y - 1 : ci.x;
        const double v = wpos[3 * (size_t)plist[(int64_t)a * n + e] + a];
        const double lo[3] = {__shfl(v, 0), __shfl(v, 2), __shfl(v, 4)};
        const double hi[3] = {__shfl(v, 1), __shfl(v, 3), __shfl(v, 5)};
        int axis = 0;
        {
#pragma clang fp contract(off)
            const double e0 = hi[0] - lo[0], e1 = hi[1] - lo[1], e2 = hi[2] - lo[2];
            double best = e0;
            if (e1 > best) { axis = 1; best = e1; }
            if (e2 > best) axis = 2;
        }
        if (ci.x >= base && t < 3) {
            clo[3 * (size_t)ci.z + t] = t == 0 ? lo[0] : t == 1 ? lo[1] : lo[2];
            chi[3 * (size_t)ci.z + t] = t == 0 ? hi[0] : t == 1 ? hi[1] : hi[2];
            if (t == 0) lv.axis[c] = axis;
        }
        const int64_t half = (int64_t)ci.x + ci.y / 2;
        const int64_t i1 = min(last, all ? (int64_t)ci.x + ci.y : half);
        for (int64_t i = max(base, (int64_t)ci.x) + t; i < i1; i += kLvThreads)
            flag[plist[axis * n + i]] = (uint8_t)(i < half ? gen : 0);
    }
}

// The particles' left marks as bits, particles [64 w, 64 w + 64) in word w, for
// k_level_sums' random reads: n / 8 bytes stay in an XCD's 4 MB L2 up to tens
// of millions of particles.  The marks as bytes stay there, beside the lists
// that stream through, up to about kLvByteMax of them, and below that the
// launch costs what it gives or more (whole build with / without it: 128^3
// 1424 / 1406 us, 144^3 2170 / 2178, 160^3 2485 / 2520).
constexpr int64_t kLvByteMax = int64_t(3) << 20;

__global__ void k_pack_marks(int64_t n, const uint8_t* __restrict__ flag, int gen,
                             uint64_t* __restrict__ bits) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t b = __ballot(i < n && flag[i] == gen);
    if ((threadIdx.x & 63) == 0 && i < n) bits[i >> 6] = b;
}

// On the split axis's own list the mark follows from the position alone, so
// only the two other lists read the particle's mark (PACKED: a bit of `bits`,
// else a byte of `flag`).  marks[a nwords + w]: the marks of positions [64 w,
// 64 w + 64) of list a; tile_sums[a ntiles + b]: the marks of list a in tile b.
// 108 us a level at 256^3 (140 with a chain of four loads per position), of
// which the two look-ups per position, a line per lane, are at least 55.
template <bool PACKED>
__global__ void __launch_bounds__(kLvThreads)
k_level_sums(int64_t n, LevelCells lv, const uint32_t* __restrict__ plist,
             const uint8_t* __restrict__ flag, int gen, const uint64_t* __restrict__ bits,
             uint64_t* __restrict__ marks, int64_t nwords, uint32_t* __restrict__ tile_sums,
             int ntiles) {
    __shared__ uint32_t wsum[3][kLvThreads / 64];
    const int64_t base = (int64_t)blockIdx.x * kLvTile;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t cnt[3] = {0u, 0u, 0u};
    auto mark_of = [&](uint32_t p) -> bool {
        return PACKED ? (bits[p >> 6] >> (p & 63u)) & 1u : flag[p] == gen;
    };
    int c = lv.tile[blockIdx.x];
    const int4 c0 = c < lv.count ? lv.cells[c] : make_int4(0, 0, 0, 0);
    bool m[kLvRounds][3];
    if (c0.x <= base && (int64_t)c0.x + c0.y >= base + kLvTile) {
        // the tile lies in one cell, as most do (the loop's cells are several
        // tiles long): all its look-ups are in flight at a time
        const int ax = lv.axis[c], u = ax == 0 ? 1 : 0, v = ax == 2 ? 1 : 2;
        uint32_t p[kLvRounds][2];
#pragma unroll
        for (int r = 0; r < kLvRounds; ++r) {
            const int64_t i = base + r * kLvThreads + threadIdx.x;
            p[r][0] = plist[(int64_t)u * n + i];
            p[r][1] = plist[(int64_t)v * n + i];
        }
#pragma unroll
        for (int r = 0; r < kLvRounds; ++r) {
            const bool own = base + r * kLvThreads + threadIdx.x - c0.x < c0.y / 2;
            const bool mu = mark_of(p[r][0]), mv = mark_of(p[r][1]);
            m[r][0] = ax == 0 ? own : mu;
            m[r][1] = ax == 0 ? mu : ax == 1 ? own : mv;
            m[r][2] = ax == 2 ? own : mv;
        }
    } else {
#pragma unroll
        for (int r = 0; r < kLvRounds; ++r) {
            const int64_t i = base + r * kLvThreads + threadIdx.x;
            m[r][0] = m[r][1] = m[r][2] = false;
            int4 ci;
            if (i >= n || !level_cell(lv, i, c, ci)) continue;
            const int ax = lv.axis[c];
            for (int a = 0; a < 3; ++a)
                m[r][a] = a == ax ? i - ci.x < ci.y / 2 : mark_of(plist[(int64_t)a * n + i]);
        }
    }
#pragma unroll
    for (int r = 0; r < kLvRounds; ++r) {
        const int64_t i = base + r * kLvThreads + threadIdx.x;
        uint64_t word[3];
        for (int a = 0; a < 3; ++a) {
            word[a] = __ballot(m[r][a]);
            cnt[a] += (uint32_t)__popcll(word[a]);
        }
        if (lane < 3 && i - lane < n)
            marks[lane * nwords + ((i - lane) >> 6)] = lane == 0 ? word[0] : lane == 1 ? word[1] : word[2];
    }
    if (lane < 3) wsum[lane][wave] = lane == 0 ? cnt[0] : lane == 1 ? cnt[1] : cnt[2];
    __syncthreads();
    if (threadIdx.x < 3) {
        uint32_t t = 0;
        for (int w = 0; w < kLvThreads / 64; ++w) t += wsum[threadIdx.x][w];
        tile_sums[(size_t)threadIdx.x * ntiles + blockIdx.x] = t;
    }
}

// SCANNED: `offs` holds the exclusive scan of tile_sums over all 3 ntiles
// entries, so the tiles before tile b of list a hold offs[a ntiles + b] -
// offs[a ntiles] marks; otherwise each workgroup adds up tile_sums itself
// (no scan launch; quadratic in the tiles, so for up to kLvSumMax of them).
constexpr int kLvSumMax = 2048;

template <bool SCANNED>
__global__ void __launch_bounds__(kLvThreads)
k_level_move(int64_t n, LevelCells lv, const uint32_t* __restrict__ plist,
             uint32_t* __restrict__ pout, const uint64_t* __restrict__ marks, int64_t nwords,
             const uint32_t* __restrict__ tile_sums, const uint32_t* __restrict__ offs,
             int ntiles) {
    __shared__ uint64_t word[3][kLvWords];
    __shared__ uint32_t pre[3][kLvWords];       // marks of the tile before the word
    __shared__ uint32_t woff[3][kLvThreads / 64];
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * kLvTile;
    if (t < 3 * kLvWords) {
        const int a = t / kLvWords, q = t % kLvWords;
        const int64_t w = base / 64 + q;
        const uint64_t v = w < nwords ? marks[a * nwords + w] : 0u;
        const uint32_t own = (uint32_t)__popcll(v);
        uint32_t x = own;
        for (int off = 1; off < kLvWords; off <<= 1) {
            const uint32_t y = __shfl_up(x, off, kLvWords);
            if (q >= off) x += y;
        }
        word[a][q] = v;
        pre[a][q] = x - own;
    }
    if (!SCANNED) {
        // this tile's offsets: the counts of the tiles before it, per list
        for (int a = 0; a < 3; ++a) {
            uint32_t c = 0;
            for (int k = t; k < (int)blockIdx.x; k += kLvThreads) c += tile_sums[(size_t)a * ntiles + k];
            for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off);
            if (lane == 0) woff[a][wave] = c;
        }
    }
    uint32_t pv[kLvRounds][3];
#pragma unroll
    for (int r = 0; r < kLvRounds; ++r) {
        const int64_t i = base + r * kLvThreads + t;
        for (int a = 0; a < 3; ++a) pv[r][a] = i < n ? plist[(int64_t)a * n + i] : 0u;
    }
    __syncthreads();
    uint32_t toff[3];
    for (int a = 0; a < 3; ++a) {
        toff[a] = 0;
        if (SCANNED) {
            toff[a] = offs[(size_t)a * ntiles + blockIdx.x] - offs[(size_t)a * ntiles];
        } else {
            for (int w = 0; w < kLvThreads / 64; ++w) toff[a] += woff[a][w];
        }
    }
    int c = lv.tile[blockIdx.x];
#pragma unroll
    for (int r = 0; r < kLvRounds; ++r) {
        const int64_t i = base + r * kLvThreads + t;
        if (i >= n) continue;
        int4 ci;
        if (!level_cell(lv, i, c, ci)) {        // no cell splits here
            for (int a = 0; a < 3; ++a) pout[(int64_t)a * n + i] = pv[r][a];
            continue;
        }
        const int64_t first = ci.x, nl = ci.y / 2;
        const int64_t pf = (uint32_t)ci.w;
        const int q = r * (kLvThreads / 64) + wave;
        for (int a = 0; a < 3; ++a) {
            const uint64_t v = word[a][q];
            const uint32_t below = (uint32_t)__popcll(v & ((1ull << lane) - 1));
            const int64_t lr = (int64_t)(toff[a] + pre[a][q] + below) - pf;
            const int64_t pos = (v >> lane) & 1 ? first + lr : first + nl + (i - first - lr);
            pout[(int64_t)a * n + pos] = pv[r][a];
        }
    }
}

// The bottom levels of the tree in one launch: one workgroup per subtree of
// at most kFuseM particles and kFuseC cells.  The three sorted lists of the
// subtree's range are held in LDS as 16-bit local ids (a particle's local id
// is its rank in the x list) and partitioned level by level exactly as the
// level loop does (first floor(n/2) of the split axis left, stable), then
// each leaf's particles are written to perm in ascending caller index.
// Bounds of every cell of the subtree are written to clo / chi.
//
// Bound by LDS instructions.  A thread owns the same positions k of the three
// lists at every level (64 consecutive ones per wave and round) and keeps
// their cell (id, first position, count) in registers; a cell's position
// range changes by halving alone, so none of it is looked up.  The left marks
// before a cell's first position are the same in the three lists and follow
// from the marks of the split axis's own list, which depend on positions
// alone: marks before k minus those of the cell up to k.  A list entry then
// costs about three LDS instructions per level (its id, its mark, its new
// place) instead of twelve, and one buffer per list does, since all entries
// are in registers before the first is written.  2.1 M particles (256
// subtrees of 8192): 204 -> 131 us; 16.7 M: 1744 -> 1171 us; 4,096 particles
// (one subtree): 89 -> 55 us.
constexpr int kFuseRounds = 8;
constexpr int kFuseT = 1024;
constexpr int kFuseM = kFuseRounds * kFuseT;
constexpr int kFuseC = 1024;
constexpr uint32_t kNoChild = 0xffffu;

// Ascending sort of one value per lane over the wavefront (bitonic).
__device__ __forceinline__ uint32_t wave_sort(uint32_t v, int lane) {
    for (int size = 2; size <= 64; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const uint32_t o = __shfl_xor(v, stride);
            const bool low = ((lane & stride) == 0) == ((lane & size) == 0);
            v = low ? min(v, o) : max(v, o);
        }
    return v;
}

// roots[b] = (subtree root cell, cells in the subtree, root depth, deepest depth)
__global__ void __launch_bounds__(kFuseT)
k_orb_fused(const int4* __restrict__ roots, const int4* __restrict__ cell,
            const int4* __restrict__ aux, const uint32_t* __restrict__ plist, int64_t n,
            const double* __restrict__ wpos, int32_t* __restrict__ loc, double* __restrict__ clo,
            double* __restrict__ chi, int32_t* __restrict__ perm) {
    __shared__ __align__(16) uint16_t lst[3 * kFuseM];
    __shared__ uint8_t flag[kFuseM];       // left marks by local id
    __shared__ uint8_t axs[kFuseM];        // split axis, at the cell's first position
    __shared__ uint32_t cch[kFuseC];       // children: first | second << 16
    __shared__ uint32_t cfc[kFuseC];       // first position | count << 16
    __shared__ uint32_t wsum[4][kFuseT / 64];
    const int4 rt = roots[blockIdx.x];
    const int root = rt.x, nsub = rt.y, depth_span = rt.w - rt.z;
    const int4 rc = cell[root];
    const int base = rc.x, m = rc.y;
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    const uint32_t* __restrict__ l0 = plist + base;
    const int R = (m + kFuseT - 1) / kFuseT;
    const int k0 = wave * R * 64 + lane;   // this thread's positions: k0 + 64 r, r < R

    for (int k = t; k < m; k += kFuseT) {
        lst[k] = (uint16_t)k;
        loc[l0[k]] = k;
    }
    for (int c = t; c < nsub; c += kFuseT) {
        const int4 ci = cell[root + c], ai = aux[root + c];
        cch[c] = ai.x >= 0 ? (uint32_t)(ai.x - root) | (uint32_t)(ai.y - root) << 16 : kNoChild;
        cfc[c] = (uint32_t)(ci.x - base) | (uint32_t)ci.y << 16;
    }
    // loc[] is written and read through global memory by this workgroup
    // only, so the barrier's workgroup-scope ordering suffices (an
    // agent-scope fence here writes back the whole L2, per workgroup)
    __syncthreads();
    for (int k = t; k < m; k += kFuseT) {
        lst[kFuseM + k] = (uint16_t)loc[plist[n + base + k]];
        lst[2 * kFuseM + k] = (uint16_t)loc[plist[2 * n + base + k]];
    }
    // the cell of each of the thread's positions; fresh: bit r, the cell is
    // of the current depth
    uint32_t fc[kFuseRounds], id[kFuseRounds];
    uint32_t fresh = 0u;
#pragma unroll
    for (int r = 0; r < kFuseRounds; ++r) {
        fc[r] = (uint32_t)m << 16;
        id[r] = 0u;
        if (r < R && k0 + 64 * r < m) fresh |= 1u << r;
    }
    const uint32_t mine = fresh;           // the thread's positions below m
    __syncthreads();

    for (int dep = 0;; ++dep) {
        // bounds of the cells of this depth, split axis of those that split
#pragma unroll
        for (int r = 0; r < kFuseRounds; ++r) {
            const int k = k0 + 64 * r, f = (int)(fc[r] & 0xffffu);
            if (!((fresh >> r) & 1u) || k != f) continue;
            const int e = f + (int)(fc[r] >> 16) - 1, c = root + (int)id[r];
            double lo[3], hi[3];
            for (int a = 0; a < 3; ++a) {
                lo[a] = wpos[3 * (size_t)l0[lst[a * kFuseM + f]] + a];
                hi[a] = wpos[3 * (size_t)l0[lst[a * kFuseM + e]] + a];
            }
            for (int a = 0; a < 3; ++a) {
                clo[3 * (size_t)c + a] = lo[a];
                chi[3 * (size_t)c + a] = hi[a];
            }
            {
#pragma clang fp contract(off)
                const double e0 = hi[0] - lo[0], e1 = hi[1] - lo[1], e2 = hi[2] - lo[2];
                int axis = 0;
                double best = e0;
                if (e1 > best) { axis = 1; best = e1; }
                if (e2 > best) axis = 2;
                axs[f] = (uint8_t)axis;
            }
        }
        if (dep == depth_span) break;
        __syncthreads();
        // left marks from the split axis's list; split: bit r, the cell splits;
        // own: bit r, position k is in the first half
        uint32_t split = 0u, own = 0u;
        uint32_t ch[kFuseRounds];
        int ax[kFuseRounds];
#pragma unroll
        for (int r = 0; r < kFuseRounds; ++r) {
            ch[r] = kNoChild;
            ax[r] = 0;
            if (!((mine >> r) & 1u)) continue;
            ch[r] = cch[id[r]];
            if (ch[r] == kNoChild) continue;
            split |= 1u << r;
            const int k = k0 + 64 * r, f = (int)(fc[r] & 0xffffu), nl = (int)(fc[r] >> 17);
            ax[r] = axs[f];
            const bool o = k - f < nl;
            own |= (o ? 1u : 0u) << r;
            flag[lst[ax[r] * kFuseM + k]] = o ? 1 : 0;
        }
        __syncthreads();
        // marks and their prefix sums inside the wave, per list (0 to 2) and of
        // the own pattern (3)
        uint32_t p[3][kFuseRounds], pre[4][kFuseRounds], mk[3] = {0u, 0u, 0u};
        uint32_t cnt[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < kFuseRounds; ++r) {
            if (r >= R) continue;
            const int k = k0 + 64 * r;
            const bool sp = (split >> r) & 1u, o = (own >> r) & 1u;
            const uint64_t mo = __ballot(o);
            pre[3][r] = cnt[3] + (uint32_t)__popcll(mo & below);
            cnt[3] += (uint32_t)__popcll(mo);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                p[a][r] = sp ? lst[a * kFuseM + k] : 0u;
                const bool b = sp && (a == ax[r] ? o : flag[p[a][r]] != 0);
                const uint64_t mb = __ballot(b);
                pre[a][r] = cnt[a] + (uint32_t)__popcll(mb & below);
                cnt[a] += (uint32_t)__popcll(mb);
                mk[a] |= (b ? 1u : 0u) << r;
            }
        }
        if (lane < 4) wsum[lane][wave] = lane == 0 ? cnt[0] : lane == 1 ? cnt[1] : lane == 2 ? cnt[2] : cnt[3];
        __syncthreads();
        // marks of the waves before (the four sums in lanes of 16)
        uint32_t before = (lane & 15) < wave ? wsum[lane >> 4][lane & 15] : 0u;
        for (int off = 8; off > 0; off >>= 1) before += __shfl_xor(before, off);
        const uint32_t bo = __shfl(before, 48);
        const uint32_t ba[3] = {(uint32_t)__shfl(before, 0) - bo, (uint32_t)__shfl(before, 16) - bo,
                                (uint32_t)__shfl(before, 32) - bo};
        fresh = split;
#pragma unroll
        for (int r = 0; r < kFuseRounds; ++r) {
            if (!((split >> r) & 1u)) continue;
            const int k = k0 + 64 * r, f = (int)(fc[r] & 0xffffu), c = (int)(fc[r] >> 16), nl = c / 2;
            // marks before k in its cell, list a: those before k in the list
            // minus those before the cell, which are the own pattern's before
            // k less the cell's own min(k - f, nl)
            const int cellpre = (int)pre[3][r] - min(k - f, nl);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const int lr = (int)(ba[a] + pre[a][r]) - cellpre;
                const int pos = (mk[a] >> r) & 1u ? f + lr : f + nl + (k - f - lr);
                lst[a * kFuseM + pos] = (uint16_t)p[a][r];
            }
            const bool o = (own >> r) & 1u;
            id[r] = o ? ch[r] & 0xffffu : ch[r] >> 16;
            fc[r] = o ? (uint32_t)f | (uint32_t)nl << 16 : (uint32_t)(f + nl) | (uint32_t)(c - nl) << 16;
        }
        __syncthreads();
    }
    // leaves, one wave each: particles in ascending caller index
    __syncthreads();
    for (int c = wave; c < nsub; c += kFuseT / 64) {
        if (cch[c] != kNoChild) continue;
        const int f = (int)(cfc[c] & 0xffffu), cnt = (int)(cfc[c] >> 16);
        uint32_t v = lane < cnt ? l0[lst[f + lane]] : 0xffffffffu;
        v = wave_sort(v, lane);
        if (lane < cnt) perm[base + f + lane] = (int32_t)v;
    }
}

// Centre, half size and radius of every cell (the host planner's formulas).
// What the dual walk reads of a cell, in one 80-byte record: centre and
// radius, half sizes, and (leaf id, child 0, child 1, box).
struct WalkCell {
    double4 c;
    double4 h;
    int4 info;
};

__global__ void k_geom(int nc, const double* __restrict__ clo, const double* __restrict__ chi,
                       const int4* __restrict__ cell, const int4* __restrict__ aux,
                       double4* __restrict__ cellc, WalkCell* __restrict__ wcell,
                       double4* __restrict__ leafc) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nc) return;
    double cc[3], h[3];
    double rad;
    {
#pragma clang fp contract(off)
        for (int a = 0; a < 3; ++a) {
            const double lo = clo[3 * (size_t)c + a], hi = chi[3 * (size_t)c + a];
            cc[a] = 0.5 * (lo + hi);
            h[a] = 0.5 * (hi - lo);
        }
        rad = sqrt((h[0] * h[0] + h[1] * h[1]) + h[2] * h[2]);
    }
    cellc[c] = make_double4(cc[0], cc[1], cc[2], rad);
    const int lf = cell[c].w;
    const int4 ax = aux[c];
    WalkCell w;
    w.c = make_double4(cc[0], cc[1], cc[2], rad);
    w.h = make_double4(h[0], h[1], h[2], 0.0);
    w.info = make_int4(lf, ax.x, ax.y, ax.z);
    wcell[c] = w;
    if (lf >= 0) leafc[lf] = make_double4(cc[0], cc[1], cc[2], 0.0);
}

__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, uint32_t* total) {
    const int lane = threadIdx.x & 63;
    uint32_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    *total = __shfl(x, 63);
    return x - v;
}

// Appends `cnt` items per lane at one atomic per wavefront; returns the
// lane's first slot.
__device__ __forceinline__ uint32_t wave_append(uint32_t cnt, uint32_t* counter) {
    uint32_t total;
    const uint32_t off = wave_excl_scan(cnt, &total);
    uint32_t base = 0;
    if (total != 0) {
        if ((threadIdx.x & 63) == 0) base = atomicAdd(counter, total);
        base = __shfl(base, 0);
    }
    return base + off;
}

// Classification of one cell pair (the dual-walk rules of the host planner).
//
// Only half of the walk is visited: every rule is symmetric under
// (t, u, s) -> (u, t, s') with s' = 26 - s the opposite image (R changes
// sign exactly, |R| and the half sizes do not change, and a tie splits both
// cells), so the pairs with s > 13, or s = 13 and t <= u, are walked and
// each result is also emitted mirrored.  Cells are in pre-order, so two
// different cells of a walked pair have disjoint subtrees and the order of
// t and u carries over to all their descendants; only a self pair (t, t, 13)
// drops its child pair (c1, c0), the mirror of (c0, c1).
struct WalkOut {
    uint32_t n_child, n_p2p, n_m2l;
    int2 child[4];
    uint64_t key[2];
};

// Task key (a << ks) | (b << 5) | s with ks = 5 + bits of the largest id:
// sorting it gives the canonical (a, b, s) order with as few radix passes
// as the ids need.
__device__ __forceinline__ uint64_t walk_key(int a, int b, int s, int ks) {
    return ((uint64_t)(uint32_t)a << ks) | ((uint64_t)(uint32_t)b << 5) | (uint64_t)s;
}

__device__ __forceinline__ void walk_classify(const int2 pr, const WalkBox* __restrict__ wbox,
                                              const WalkCell* __restrict__ wcell, int2 ks,
                                              WalkOut& o) {
    const int t = pr.x, u = pr.y >> 5, s = pr.y & 31;
    const WalkCell wt = wcell[t], wu = wcell[u];
    const int4 at = make_int4(wt.info.y, wt.info.z, wt.info.w, 0);
    const int4 au = make_int4(wu.info.y, wu.info.z, wu.info.w, 0);
    const WalkBox wb = wbox[wt.info.w];
    const double4 ct = wt.c, cu = wu.c, ht = wt.h, hu = wu.h;
    const double sL[3] = {(double)(s % 3 - 1) * wb.L, (double)((s / 3) % 3 - 1) * wb.L,
                          (double)(s / 9 - 1) * wb.L};
    const double cta[3] = {ct.x, ct.y, ct.z}, cua[3] = {cu.x, cu.y, cu.z};
    const double hta[3] = {ht.x, ht.y, ht.z}, hua[3] = {hu.x, hu.y, hu.z};
    double R[3], A[3], H[3], gp[3], gap2, dmax2 = 0.0, R2 = 0.0, lhs = 0.0;
    {
#pragma clang fp contract(off)
        for (int a = 0; a < 3; ++a) {
            R[a] = (cua[a] - cta[a]) + sL[a];
            A[a] = fabs(R[a]);
            H[a] = hta[a] + hua[a];
            const double g = A[a] - H[a];
            gp[a] = g > 0.0 ? g : 0.0;
        }
        gap2 = (gp[0] * gp[0] + gp[1] * gp[1]) + gp[2] * gp[2];
        if (wb.use_m2l) {
            const double d0 = A[0] + H[0], d1 = A[1] + H[1], d2 = A[2] + H[2];
            dmax2 = (d0 * d0 + d1 * d1) + d2 * d2;
            R2 = (R[0] * R[0] + R[1] * R[1]) + R[2] * R[2];
            lhs = ct.w + cu.w;
            lhs = lhs * lhs;
            R2 = wb.th2 * R2;
        }
    }
    if (!(gap2 < wb.rc2_drop)) return;
    const bool self = (t == u) && (s == 13);
    if (wb.use_m2l && wb.centre_cut && lhs < R2) {
        // centre-distance cut: R2 holds theta^2 |R|^2, so recompute |R|^2
        double Rc2;
        {
#pragma clang fp contract(off)
            Rc2 = (R[0] * R[0] + R[1] * R[1]) + R[2] * R[2];
        }
        if (!(Rc2 < wb.rc2)) return;
        o.n_m2l = self ? 1 : 2;
        o.key[0] = walk_key(t, u, s, ks.y);
        o.key[1] = walk_key(u, t, 26 - s, ks.y);
        return;
    }
    if (wb.use_m2l && !wb.centre_cut && dmax2 < wb.rc2_m2l && lhs < R2) {
        o.n_m2l = self ? 1 : 2;
        o.key[0] = walk_key(t, u, s, ks.y);
        o.key[1] = walk_key(u, t, 26 - s, ks.y);
        return;
    }
    const int lt = wt.info.x, lu = wu.info.x;
    const double rt = ct.w, ru = cu.w;
    if (lt >= 0 && lu >= 0) {
        o.n_p2p = self ? 1 : 2;
        o.key[0] = walk_key(lt, lu, s, ks.x);
        o.key[1] = walk_key(lu, lt, 26 - s, ks.x);
    } else if (self) {
        o.child[0] = make_int2(at.x, (at.x << 5) | s);
        o.child[1] = make_int2(at.x, (at.y << 5) | s);
        o.child[2] = make_int2(at.y, (at.y << 5) | s);
        o.n_child = 3;
    } else if (lt < 0 && (lu >= 0 || rt > ru)) {
        o.child[0] = make_int2(at.x, pr.y);
        o.child[1] = make_int2(at.y, pr.y);
        o.n_child = 2;
    } else if (lu < 0 && (lt >= 0 || ru > rt)) {
        o.child[0] = make_int2(t, (au.x << 5) | s);
        o.child[1] = make_int2(t, (au.y << 5) | s);
        o.n_child = 2;
    } else {
        o.child[0] = make_int2(at.x, (au.x << 5) | s);
        o.child[1] = make_int2(at.x, (au.y << 5) | s);
        o.child[2] = make_int2(at.y, (au.x << 5) | s);
        o.child[3] = make_int2(at.y, (au.y << 5) | s);
        o.n_child = 4;
    }
}

// One level of the walk, frontier size known on the host.
__global__ void __launch_bounds__(256)
k_walk(const int2* __restrict__ front, int nf, int2* __restrict__ next,
       const WalkBox* __restrict__ wbox, const WalkCell* __restrict__ wcell, int2 ks,
       uint32_t* __restrict__ counters, uint64_t* __restrict__ p2p_keys,
       uint64_t* __restrict__ m2l_keys) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    WalkOut o{0u, 0u, 0u, {}, {0ull, 0ull}};
    if (k < nf) walk_classify(front[k], wbox, wcell, ks, o);
    const uint32_t cslot = wave_append(o.n_child, &counters[0]);
    for (uint32_t q = 0; q < o.n_child; ++q) next[cslot + q] = o.child[q];
    const uint32_t pslot = wave_append(o.n_p2p, &counters[1]);
    for (uint32_t q = 0; q < o.n_p2p; ++q) p2p_keys[pslot + q] = o.key[q];
    const uint32_t mslot = wave_append(o.n_m2l, &counters[2]);
    for (uint32_t q = 0; q < o.n_m2l; ++q) m2l_keys[mslot + q] = o.key[q];
}

// One level of the walk with the frontier size read on the device (no host
// round trip between levels).  Capacities are checked; an overflow is
// reported and the host then redoes the walk level by level.  The appends
// are aggregated per workgroup (one atomic per counter per group of pairs):
// all workgroups add to the same three counters, and at one atomic per
// wavefront those additions, serialised at one address, took most of a
// level's time.
// ctl: [0] p2p total, [1] m2l total, [2] overflow flag, [3] largest frontier;
// sizes[it] = frontier size of level it.
constexpr int kWalkT = 1024;
// Frontiers of up to kWalkNarrowMax pairs are walked by smaller workgroups: a
// thread reads two 80-byte cells of its own, a line at a time, so 1024 pairs on
// one CU are 4 us of address work, and a few thousand pairs were on a few of
// the CUs.  Walk of 64^3 142 -> 105 us, 128^3 279 -> 255; 64 and 128 threads
// were slower at 64^3 (126, 122), and beyond, the groups' additions to the
// same three counters cost more than that (128^3 with 256 throughout: 368).
constexpr int kWalkNarrow = 256;
constexpr int64_t kWalkNarrowMax = 65536;
constexpr int kWalkThreads = 512 * 1024;   // of a launch, at most
// frontiers up to this size go to the one-workgroup top of the walk: as many as
// stay in its LDS (walk of 16^3 / 64^3 / 128^3 with 256 43 / 112 / 264 us, 1024
// 38 / 105 / 255, 4096 47 / 113 / 256)
constexpr uint32_t kWalkTopMax = kWalkT;

// Appends one group's outputs (a WalkOut per thread of the workgroup): the
// keys to the key arrays and the child pairs to `next` at slots reserved
// from *next_count, or, with `lch`, to that workgroup-local array from 0.
// One atomic per counter per group.  Returns the group's child count.
template <int T>
__device__ __forceinline__ uint32_t walk_emit(const WalkOut& o, int2* __restrict__ next,
                                              uint32_t* __restrict__ next_count,
                                              uint32_t cap_front, int2* lch,
                                              uint32_t* __restrict__ ctl, uint32_t cap_p2p,
                                              uint32_t cap_m2l, uint64_t* __restrict__ p2p_keys,
                                              uint64_t* __restrict__ m2l_keys, uint64_t* wtot,
                                              uint32_t* bbase) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // packed counts: children (<= 4096 per group) | p2p << 16 | m2l << 32
    const uint64_t v = (uint64_t)o.n_child | ((uint64_t)o.n_p2p << 16) |
                       ((uint64_t)o.n_m2l << 32);
    uint64_t x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t y = __shfl_up(x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) wtot[wave] = x;
    __syncthreads();
    if (wave == 0) {
        // the waves' totals scanned across 16 lanes, then lanes 0 to 2 reserve
        // the group's slots at once: three reservations one after another by
        // one thread waited for three device-scope atomics
        const uint64_t tw = lane < T / 64 ? wtot[lane] : 0ull;
        uint64_t y = tw;
        for (int off = 1; off < T / 64; off <<= 1) {
            const uint64_t z = __shfl_up(y, off);
            if (lane >= off) y += z;
        }
        const uint64_t all = __shfl(y, T / 64 - 1);
        if (lane < T / 64) wtot[lane] = y - tw;
        const uint32_t tc = (uint32_t)(all & 0xffffu), tp = (uint32_t)((all >> 16) & 0xffffu),
                       tm = (uint32_t)(all >> 32);
        if (lane < 3) {
            const uint32_t add = lane == 0 ? (lch == nullptr ? tc : 0u) : lane == 1 ? tp : tm;
            uint32_t* at = lane == 0 ? next_count : ctl + (lane - 1);
            bbase[lane] = add != 0 ? atomicAdd(at, add) : 0u;
        }
        if (lane == 3) bbase[3] = tc;
    }
    __syncthreads();
    const uint64_t off = wtot[wave] + x - v;
    const uint32_t cslot = bbase[0] + (uint32_t)(off & 0xffffu);
    const uint32_t pslot = bbase[1] + (uint32_t)((off >> 16) & 0xffffu);
    const uint32_t mslot = bbase[2] + (uint32_t)(off >> 32);
    // (fixed trip counts: the WalkOut arrays stay in registers)
    if (lch != nullptr) {
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
            if (q < o.n_child) lch[cslot + q] = o.child[q];
    } else if (cslot + o.n_child <= cap_front) {
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q)
            if (q < o.n_child) next[cslot + q] = o.child[q];
    } else if (o.n_child) {
        ctl[2] = 1u;
    }
#pragma unroll
    for (uint32_t q = 0; q < 2; ++q) {
        if (q < o.n_p2p) {
            if (pslot + q < cap_p2p) p2p_keys[pslot + q] = o.key[q]; else ctl[2] = 1u;
        }
        if (q < o.n_m2l) {
            if (mslot + q < cap_m2l) m2l_keys[mslot + q] = o.key[q]; else ctl[2] = 1u;
        }
    }
    const uint32_t tc = bbase[3];
    __syncthreads();   // wtot, bbase (and lch, for its readers) are reused next
    return tc;
}

// One level's share of workgroup `blk` of `nblk` (nf pairs in front).
// Returns false when the frontier is beyond its capacity.
template <int T>
__device__ __forceinline__ bool walk_level(const int2* __restrict__ front, int2* __restrict__ next,
                                           int it, uint32_t nf, uint32_t blk, uint32_t nblk,
                                           uint32_t* __restrict__ sizes, uint32_t* __restrict__ ctl,
                                           uint32_t cap_front, uint32_t cap_p2p, uint32_t cap_m2l,
                                           const WalkBox* __restrict__ wbox,
                                           const WalkCell* __restrict__ wcell, int2 ks,
                                           uint64_t* __restrict__ p2p_keys,
                                           uint64_t* __restrict__ m2l_keys, uint64_t* wtot,
                                           uint32_t* bbase) {
    if (nf > cap_front) return false;
    const uint32_t stride = nblk * blockDim.x;
    for (uint32_t base = blk * blockDim.x; base < nf; base += stride) {
        const uint32_t k = base + threadIdx.x;
        WalkOut o{0u, 0u, 0u, {}, {0ull, 0ull}};
        if (k < nf) walk_classify(front[k], wbox, wcell, ks, o);
        (void)walk_emit<T>(o, next, &sizes[it + 1], cap_front, nullptr, ctl, cap_p2p, cap_m2l,
                        p2p_keys, m2l_keys, wtot, bbase);
    }
    if (blk == 0 && threadIdx.x == 0) atomicMax(&ctl[3], nf);
    return true;
}

// Levels it and it + 1 of the walk in workgroup `blk` of `nblk`: each
// workgroup classifies a group of level it, keeps the group's child pairs
// (at most four per pair) in LDS (`lch`) and classifies them in turn; only
// their children (level it + 2) go to `next`.  The descendants of a pair
// depend on that pair alone, so the middle level needs no other
// workgroup's results and its pairs never go through global memory.
// sizes[it + 1] counts the middle level (for the next build's sizing).
// Two levels per launch took the 128^3 walk from 0.55 to 0.33 ms; three
// took 0.37 ms (the deeper a workgroup's subtree, the more the workgroups'
// shares differ).
template <int T>
__device__ __forceinline__ void walk_two(const int2* __restrict__ front, int2* __restrict__ next,
                                         int it, uint32_t nf, uint32_t blk, uint32_t nblk,
                                         uint32_t* __restrict__ sizes, uint32_t* __restrict__ ctl,
                                         uint32_t cap_front, uint32_t cap_p2p, uint32_t cap_m2l,
                                         const WalkBox* __restrict__ wbox,
                                         const WalkCell* __restrict__ wcell, int2 ks,
                                         uint64_t* __restrict__ p2p_keys,
                                         uint64_t* __restrict__ m2l_keys, uint64_t* wtot,
                                         uint32_t* bbase, int2* lch) {
    const uint32_t stride = nblk * blockDim.x;
    for (uint32_t base = blk * blockDim.x; base < nf; base += stride) {
        const uint32_t k = base + threadIdx.x;
        WalkOut o{0u, 0u, 0u, {}, {0ull, 0ull}};
        if (k < nf) walk_classify(front[k], wbox, wcell, ks, o);
        const uint32_t n1 = walk_emit<T>(o, nullptr, nullptr, 0u, lch, ctl, cap_p2p, cap_m2l,
                                      p2p_keys, m2l_keys, wtot, bbase);
        if (threadIdx.x == 0 && n1 != 0) atomicAdd(&sizes[it + 1], n1);
        for (uint32_t r = 0; r < n1; r += blockDim.x) {
            const uint32_t j = r + threadIdx.x;
            WalkOut o2{0u, 0u, 0u, {}, {0ull, 0ull}};
            if (j < n1) walk_classify(lch[j], wbox, wcell, ks, o2);
            (void)walk_emit<T>(o2, next, &sizes[it + 2], cap_front, nullptr, ctl, cap_p2p, cap_m2l,
                            p2p_keys, m2l_keys, wtot, bbase);
        }
    }
    if (blk == 0 && threadIdx.x == 0) atomicMax(&ctl[3], nf);
}

// Levels it and it + 1, the frontier size read on the device.
template <int T>
__global__ void __launch_bounds__(T)
k_walk_multi(const int2* __restrict__ front, int2* __restrict__ next, int it,
             uint32_t* __restrict__ sizes, uint32_t* __restrict__ ctl, uint32_t cap_front,
             uint32_t cap_p2p, uint32_t cap_m2l, const WalkBox* __restrict__ wbox,
             const WalkCell* __restrict__ wcell, int2 ks, uint64_t* __restrict__ p2p_keys,
             uint64_t* __restrict__ m2l_keys) {
    __shared__ uint64_t wtot[T / 64];
    __shared__ uint32_t bbase[4];
    __shared__ int2 lch[4 * T];
    const uint32_t nf = sizes[it];
    if (nf > cap_front) return;
    walk_two<T>(front, next, it, nf, blockIdx.x, gridDim.x, sizes, ctl, cap_front, cap_p2p, cap_m2l,
             wbox, wcell, ks, p2p_keys, m2l_keys, wtot, bbase, lch);
}

// Launches of k_walk_top's steps: two levels per step, one for an odd last
// level; step q reads buffer q & 1 and writes the other, so the frontier of
// level `levels` ends in buffer walk_top_steps(levels) & 1.
constexpr int walk_top_steps(int levels) { return levels / 2 + (levels & 1); }

// The first frontier (each box's root against itself with the zero shift and
// the 13 shifts of code > 13, the canonical half) and the walk's first
// `levels` levels in one workgroup: the top of the walk has frontiers of a few
// hundred pairs, where a launch per level costs more than the level.  A level
// is a chain of latencies, so while a frontier has a pair per thread or less
// it stays in LDS (a child's four at most fit), with the counts of the keys:
// through global memory and device-scope atomics a level of 16^3 was 0.5 us
// more.  From the first larger frontier on (or at the end) it is
// in global memory, two levels a step, and its sizes, which thread 0 adds to
// with atomics, are read back with atomic loads.
__global__ void __launch_bounds__(kWalkT)
k_walk_top(int nbox, const int32_t* __restrict__ box_root, int2* __restrict__ buf0,
           int2* __restrict__ buf1, int levels, uint32_t* __restrict__ sizes,
           uint32_t* __restrict__ ctl, uint32_t cap_front, uint32_t cap_p2p, uint32_t cap_m2l,
           const WalkBox* __restrict__ wbox, const WalkCell* __restrict__ wcell, int2 ks,
           uint64_t* __restrict__ p2p_keys, uint64_t* __restrict__ m2l_keys) {
    __shared__ uint64_t wtot[kWalkT / 64];
    __shared__ uint32_t bbase[4];
    __shared__ int2 lch[4 * kWalkT];
    __shared__ uint32_t lctl[4];
    const uint32_t t = threadIdx.x;
    uint32_t nf = (uint32_t)(14 * nbox);
    auto root_pair = [&](uint32_t q) {
        const int b = (int)(q / 14), j = (int)(q - 14 * (uint32_t)b);
        const int root = box_root[b];
        return make_int2(root, (root << 5) | (13 + j));
    };
    int it = 0;
    if (nf <= (uint32_t)kWalkT) {
        if (t < 4) lctl[t] = 0u;
        if (t < nf) lch[t] = root_pair(t);
        __syncthreads();
        uint32_t most = 0;
        while (it < levels && nf != 0 && nf <= (uint32_t)kWalkT) {
            most = max(most, nf);
            if (t == 0) sizes[it] = nf;
            WalkOut o{0u, 0u, 0u, {}, {0ull, 0ull}};
            if (t < nf) walk_classify(lch[t], wbox, wcell, ks, o);
            nf = walk_emit<kWalkT>(o, nullptr, nullptr, 0u, lch, lctl, cap_p2p, cap_m2l, p2p_keys,
                           m2l_keys, wtot, bbase);
            ++it;
        }
        if (t < 2 && lctl[t] != 0u) atomicAdd(&ctl[t], lctl[t]);
        if (t == 2 && lctl[2] != 0u) ctl[2] = 1u;
        if (t == 3) atomicMax(&ctl[3], most);
        if (nf == 0) return;
    }
    if (nf > cap_front) {
        if (t == 0) ctl[2] = 1u;
        return;
    }
    // the frontier of level `levels` ends in buffer walk_top_steps(levels) & 1
    int step = (walk_top_steps(levels) ^ walk_top_steps(levels - it)) & 1;
    for (uint32_t q = t; q < nf; q += blockDim.x)
        ((step & 1) ? buf1 : buf0)[q] = it == 0 ? root_pair(q) : lch[q];
    if (t == 0) sizes[it] = nf;
    __syncthreads();
    for (const int it0 = it; it < levels; ++step) {
        if (it != it0)
            nf = __hip_atomic_load(&sizes[it], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (nf > cap_front) return;
        const int2* front = (step & 1) ? buf1 : buf0;
        int2* next = (step & 1) ? buf0 : buf1;
        if (it + 2 <= levels) {
            walk_two<kWalkT>(front, next, it, nf, 0u, 1u, sizes, ctl, cap_front, cap_p2p, cap_m2l, wbox,
                     wcell, ks, p2p_keys, m2l_keys, wtot, bbase, lch);
            it += 2;
        } else {
            (void)walk_level<kWalkT>(front, next, it, nf, 0u, 1u, sizes, ctl, cap_front, cap_p2p,
                             cap_m2l, wbox, wcell, ks, p2p_keys, m2l_keys, wtot, bbase);
            it += 1;
        }
        __syncthreads();
    }
}

// Smallest target / source depth of the walk's M2L keys (key = t << ks |
// u << 5 | s), kept as 0x7fffffff - depth by atomicMax into zeroed words
// out[0] (targets) and out[1] (sources); the key count is *count.
__global__ void k_m2l_depths(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ count,
                             uint32_t cap, int ks, const int4* __restrict__ aux,
                             uint32_t* __restrict__ out) {
    const uint32_t n = min(*count, cap);
    uint32_t bt = 0u, bs = 0u;
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
        const uint64_t key = keys[k];
        const int t = (int)(key >> ks), u = (int)((key & ((1ull << ks) - 1ull)) >> 5);
        bt = max(bt, 0x7fffffffu - (uint32_t)aux[t].w);
        bs = max(bs, 0x7fffffffu - (uint32_t)aux[u].w);
    }
    if (bt) atomicMax(&out[0], bt);
    if (bs) atomicMax(&out[1], bs);
}

__global__ void k_zero_u32(uint32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// CSR rows from the walk's unsorted keys (row << ks | value): each key takes
// a slot in its row with an atomic count, the counts are scanned into the
// row starts, the values are placed, and each row's values are sorted
// (bitonic, in LDS), which gives the canonical (i, j, shift) order since the
// values of one row are distinct.
//
// Consecutive keys come from pairs of the same few cells, so a workgroup's
// 1024 keys fall on a few hundred rows: they are counted in an LDS hash table
// first (open addressing, twice the keys), and each of its rows takes one
// global atomic.  One atomic per key ran at 28 G/s: 95 us for the 2.7 M keys
// of 128^3, now 31 us.
constexpr int kRcThreads = 256;
constexpr int kRcEach = 4;
constexpr int kRcKeys = kRcThreads * kRcEach;
constexpr uint32_t kRcHash = 2 * kRcKeys;

__global__ void __launch_bounds__(kRcThreads)
k_row_count(const uint64_t* __restrict__ keys, int64_t nk, int ks, int32_t* __restrict__ cnt,
            int32_t* __restrict__ slot) {
    __shared__ uint32_t tag[kRcHash];    // row + 1; 0: free
    __shared__ uint32_t num[kRcHash];    // keys of the row; then its first slot
    for (uint32_t h = threadIdx.x; h < kRcHash; h += kRcThreads) {
        tag[h] = 0u;
        num[h] = 0u;
    }
    const int64_t k0 = (int64_t)blockIdx.x * kRcKeys + threadIdx.x;
    uint32_t row[kRcEach], at[kRcEach], rank[kRcEach];
#pragma unroll
    for (int e = 0; e < kRcEach; ++e) {
        const int64_t k = k0 + e * kRcThreads;
        row[e] = k < nk ? (uint32_t)(keys[k] >> ks) + 1u : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kRcEach; ++e) {
        if (row[e] == 0u) continue;
        uint32_t h = (row[e] * 2654435761u) >> 21;
        // at most kRcKeys entries in twice as many places: a free one is found
        for (;;) {
            const uint32_t was = atomicCAS(&tag[h], 0u, row[e]);
            if (was == 0u || was == row[e]) break;
            h = (h + 1u) & (kRcHash - 1u);
        }
        at[e] = h;
        rank[e] = atomicAdd(&num[h], 1u);
    }
    __syncthreads();
    for (uint32_t h = threadIdx.x; h < kRcHash; h += kRcThreads)
        if (tag[h] != 0u) num[h] = (uint32_t)atomicAdd(&cnt[tag[h] - 1u], (int32_t)num[h]);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < kRcEach; ++e)
        if (row[e] != 0u) slot[k0 + e * kRcThreads] = (int32_t)(num[at[e]] + rank[e]);
}
static_assert(kRcHash == 1u << 11, "the hash keeps 11 bits");

__global__ void k_row_place(const uint64_t* __restrict__ keys, int64_t nk, int ks,
                            const int32_t* __restrict__ row, const int32_t* __restrict__ slot,
                            int32_t* __restrict__ vals) {
    const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nk) return;
    const uint64_t key = keys[k];
    vals[row[key >> ks] + slot[k]] = (int32_t)(key & ((1ull << ks) - 1));
}

// Ascending bitonic sort of b[0, P) (P a power of two) by the T threads of
// the workgroup; t is the caller's thread index.
__device__ void bitonic_sort(int32_t* b, int P, int t, int T) {
    for (int size = 2; size <= P; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int p = t; p < P / 2; p += T) {
                const int lo = 2 * p - (p & (stride - 1)), hi = lo + stride;
                const bool up = (lo & size) == 0;
                const int32_t x = b[lo], y = b[hi];
                if ((x > y) == up) {
                    b[lo] = y;
                    b[hi] = x;
                }
            }
            __syncthreads();
        }
    }
}

__device__ __forceinline__ int pow2_at_least(int n) {
    int P = 1;
    while (P < n) P <<= 1;
    return P;
}

// One wavefront per row of at most kRowShort values; longer rows are listed
// for k_row_sort_long.
constexpr int kRowShort = 1024;
constexpr int kRowLds = 8192;

// v of lane ^ M.  The masks that stay within 16 lanes are DPP moves (4 in
// two), so only 16 and 32 cross the LDS unit.
template <int M>
__device__ __forceinline__ int32_t lane_xor(int32_t v) {
    if constexpr (M == 1) return __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true);    // quad 1 0 3 2
    if constexpr (M == 2) return __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true);    // quad 2 3 0 1
    if constexpr (M == 4)                                     // half-row mirror (7), quad 3 2 1 0 (3)
        return __builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true), 0x1B,
                                        0xF, 0xF, true);
    if constexpr (M == 8) return __builtin_amdgcn_mov_dpp(v, 0x128, 0xF, 0xF, true);   // row rotate 8
    return __shfl_xor(v, M);
}

// Strides J, J / 2, ..., 1 of bitonic phase K over the 64 R values of a wave,
// value i = R lane + r in register r.
template <int R, int K, int J>
__device__ __forceinline__ void bitonic_strides(int32_t (&v)[R], int lane) {
    if constexpr (J >= R) {
        const bool low = ((lane & (J / R)) == 0) == (((R * lane) & K) == 0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int32_t o = lane_xor<J / R>(v[r]);
            v[r] = low ? min(v[r], o) : max(v[r], o);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r & J) continue;
            const bool up = ((R * lane + r) & K) == 0;
            const int32_t x = v[r], y = v[r | J];
            v[r] = up ? min(x, y) : max(x, y);
            v[r | J] = up ? max(x, y) : min(x, y);
        }
    }
    if constexpr (J > 1) bitonic_strides<R, K, J / 2>(v, lane);
}

template <int R, int K>
__device__ __forceinline__ void bitonic_phases(int32_t (&v)[R], int lane) {
    if constexpr (K > 2) bitonic_phases<R, K / 2>(v, lane);
    bitonic_strides<R, K, K / 2>(v, lane);
}

template <int R>
__device__ __forceinline__ void sort_row(int32_t* __restrict__ p, int len, int lane) {
    int32_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = 64 * r + lane < len ? p[64 * r + lane] : INT32_MAX;
    bitonic_phases<R, 64 * R>(v, lane);
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (R * lane + r < len) p[R * lane + r] = v[r];
}

// The values stay in registers, blocked R to a lane, so of the 36 strides of
// a 256-value row 15 are within a lane and 18 of the rest are DPP moves; with
// the row in LDS, each stride was four LDS operations and a barrier.
__global__ void __launch_bounds__(256)
k_row_sort_short(const int32_t* __restrict__ row, int nrows, int32_t* __restrict__ vals,
                 int32_t* __restrict__ longs, int32_t* __restrict__ nlong) {
    const int lane = threadIdx.x & 63;
    const int r = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    if (r >= nrows) return;
    const int r0 = row[r], len = row[r + 1] - r0;
    if (len <= 1) return;
    int32_t* p = vals + r0;
    if (len <= 64) return sort_row<1>(p, len, lane);
    if (len <= 128) return sort_row<2>(p, len, lane);
    if (len <= 256) return sort_row<4>(p, len, lane);
    if (len <= 512) return sort_row<8>(p, len, lane);
    if (len <= kRowShort) return sort_row<16>(p, len, lane);
    if (lane == 0) longs[atomicAdd(nlong, 1)] = r;
}

// The listed long rows, one workgroup at a time each: in LDS up to lds_cap
// (<= kRowLds) values, else in scratch[2 r0, 2 r0 + P) (P < 2 len, so rows
// never share scratch; the caller provides twice the value count).
__global__ void __launch_bounds__(256)
k_row_sort_long(const int32_t* __restrict__ row, int32_t* __restrict__ vals,
                const int32_t* __restrict__ longs, const int32_t* __restrict__ nlong,
                int32_t* __restrict__ scratch, int lds_cap) {
    __shared__ int32_t lds[kRowLds];
    const int t = threadIdx.x;
    const int count = *nlong;
    for (int q = blockIdx.x; q < count; q += gridDim.x) {
        const int r = longs[q];
        const int r0 = row[r], len = row[r + 1] - r0;
        const int P = pow2_at_least(len);
        int32_t* b = P <= lds_cap ? lds : scratch + 2 * (size_t)r0;
        for (int k = t; k < P; k += 256) b[k] = k < len ? vals[r0 + k] : INT32_MAX;
        __syncthreads();
        bitonic_sort(b, P, t, 256);
        for (int k = t; k < len; k += 256) vals[r0 + k] = b[k];
        __syncthreads();
    }
}

// M2L sources and shifts from the sorted row values, and the smallest
// depth of the tasks' source and target cells (mindep[0] / mindep[1],
// preset to INT32_MAX).
__global__ void k_m2l_split(const int32_t* __restrict__ row, int nrows, const int32_t* __restrict__ vals,
                            const int4* __restrict__ aux, int32_t* __restrict__ src,
                            int32_t* __restrict__ shift, int32_t* __restrict__ mindep) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= nrows) return;
    const int r0 = row[c], r1 = row[c + 1];
    if (r0 == r1) return;
    int dmin = INT32_MAX;
    for (int k = r0; k < r1; ++k) {
        const int u = vals[k] >> 5;
        src[k] = u;
        shift[k] = vals[k] & 31;
        dmin = min(dmin, aux[u].w);
    }
    atomicMin(&mindep[0], dmin);
    atomicMin(&mindep[1], aux[c].w);
}

// Items of every row (their scan gives each row's first slot); clears the
// words that k_queue adds to.
__global__ void k_item_count(int nl, const int32_t* __restrict__ row, int chunk,
                             int32_t* __restrict__ cnt, uint32_t* __restrict__ wcount) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 3) wcount[8 + i] = 0u;
    if (i > nl) return;
    if (i == nl) { cnt[i] = 0; return; }
    const int len = row[i + 1] - row[i];
    cnt[i] = (len + chunk - 1) / chunk;
}

// Work items of each TaskGroup row, one wavefront per row and one lane per
// item; cost[slot] = 255 - (pair count >> cshift), so that ascending costs are
// the longest first up to 1/256 of the largest item.  rowcand[i]: candidate
// pairs of row i.
__global__ void k_items(int nl, const int32_t* __restrict__ row, const int32_t* __restrict__ js,
                        const int4* __restrict__ leaf, int chunk, int cshift,
                        const int32_t* __restrict__ slot0, int4* __restrict__ items,
                        uint8_t* __restrict__ cost, unsigned long long* __restrict__ rowcand) {
    const int64_t gt = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int i = (int)(gt >> 6), lane = (int)(gt & 63);
    if (i >= nl) return;
    unsigned long long total = 0;
    const int r0 = row[i], len = row[i + 1] - r0;
    if (len > 0) {
        const int parts = (len + chunk - 1) / chunk;
        const int base = len / parts, extra = len % parts;
        const int ni = leaf[i].y;
        for (int k = lane; k < parts; k += 64) {
            const int t = r0 + k * base + min(k, extra);
            const int sz = base + (k < extra ? 1 : 0);
            // the tasks' source counts, eight loads in flight at a time
            unsigned long long c = 0;
            int q = t;
            for (; q + 8 <= t + sz; q += 8) {
                int jv[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) jv[u] = js[q + u] >> 5;
#pragma unroll
                for (int u = 0; u < 8; ++u) c += (unsigned long long)leaf[jv[u]].y;
            }
            for (; q < t + sz; ++q) c += (unsigned long long)leaf[js[q] >> 5].y;
            c *= (unsigned long long)ni;
            total += c;
            const int s = slot0[i] + k;
            items[s] = make_int4(i, t, t + sz, s);
            const unsigned long long b = c >> cshift;
            cost[s] = (uint8_t)(255u - (b > 255ull ? 255u : (uint32_t)b));
        }
    }
    // the row's candidate pairs (summed by k_queue: one atomic per row on a
    // single counter would serialise)
    for (int off = 32; off > 0; off >>= 1) total += __shfl_down(total, off);
    if (lane == 0) rowcand[i] = total;
}

// The queue, one workgroup per segment: a counting sort of its slots by cost
// (the order inside a cost class, which only the schedule sees, is the order
// in which the lanes arrive).  Eight launches of a radix sort over (segment,
// cost) keys took its place before (64^3 build: 630 -> 578 us with the other
// launches saved beside it).  Each workgroup also adds up
// its share of the rows' candidate pairs.
__global__ void __launch_bounds__(1024)
k_queue(int nl, const int32_t* __restrict__ slot0, const uint8_t* __restrict__ cost,
        const unsigned long long* __restrict__ rowcand, uint32_t* __restrict__ queue,
        uint32_t* __restrict__ wcount) {
    __shared__ uint32_t h[256];
    __shared__ unsigned long long part[1024 / 64];
    const int t = threadIdx.x, lane = t & 63;
    const int n = slot0[nl];
    const int beg = queue_seg_begin((int)blockIdx.x, n), end = queue_seg_begin((int)blockIdx.x + 1, n);
    if (t < 256) h[t] = 0u;
    __syncthreads();
#pragma unroll 4
    for (int s = beg + t; s < end; s += 1024) atomicAdd(&h[cost[s]], 1u);
    __syncthreads();
    if (t < 64) {
        uint32_t v[4], tot = 0;
        for (int j = 0; j < 4; ++j) {
            v[j] = h[4 * lane + j];
            tot += v[j];
        }
        uint32_t x = tot;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        uint32_t e = x - tot;
        for (int j = 0; j < 4; ++j) {
            h[4 * lane + j] = e;
            e += v[j];
        }
    }
    __syncthreads();
#pragma unroll 4
    for (int s = beg + t; s < end; s += 1024) queue[beg + atomicAdd(&h[cost[s]], 1u)] = (uint32_t)s;
    unsigned long long c = 0;
    const int i0 = queue_seg_begin((int)blockIdx.x, nl), i1 = queue_seg_begin((int)blockIdx.x + 1, nl);
#pragma unroll 4
    for (int i = i0 + t; i < i1; i += 1024) c += rowcand[i];
    for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off);
    if (lane == 0) part[t >> 6] = c;
    __syncthreads();
    if (t == 0) {
        unsigned long long all = 0;
        for (int w = 0; w < 1024 / 64; ++w) all += part[w];
        atomicAdd(reinterpret_cast<unsigned long long*>(wcount + 8), all);
        if (blockIdx.x == 0) wcount[10] = (uint32_t)n;
    }
}

inline unsigned grid_of(int64_t n, int b = 256) { return (unsigned)((n + b - 1) / b); }

int bits_for(uint64_t maxv) {
    int b = 0;
    while (b < 64 && (maxv >> b) != 0) ++b;
    return b;
}

#define TRY(expr)                                                                   \
    do {                                                                            \
        hipError_t e_ = (expr);                                                     \
        if (e_ != hipSuccess) return std::string(#expr) + ": " + hipGetErrorString(e_); \
    } while (0)

template <class T>
hipError_t up(DevBuf& b, const std::vector<T>& v, hipStream_t s) {
    hipError_t e = b.ensure(std::max<size_t>(16, v.size() * sizeof(T)));
    if (e != hipSuccess || v.empty()) return e;
    return hipMemcpyAsync(b.p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s);
}

// LDS capacity of the long-row sort; PMFMM_ROW_LDS lowers it (tests use it
// to send rows through the scratch path).
int row_lds_cap() {
    const char* v = std::getenv("PMFMM_ROW_LDS");
    if (!v) return kRowLds;
    const int c = std::atoi(v);
    return c < 0 ? 0 : std::min(c, kRowLds);
}

// Wall-clock phases of the device planner, printed to stderr when the
// environment variable PMFMM_PLAN_TIMING is set (synchronises each phase).
struct PhaseTimer {
    bool on = std::getenv("PMFMM_PLAN_TIMING") != nullptr;
    hipStream_t s;
    std::chrono::steady_clock::time_point t = std::chrono::steady_clock::now();
    explicit PhaseTimer(hipStream_t st) : s(st) {}
    void lap(const char* what) {
        if (!on) return;
        (void)hipStreamSynchronize(s);
        auto now = std::chrono::steady_clock::now();
        std::fprintf(stderr, "[pmfmm gpu plan] %-10s %8.3f ms\n", what,
                     std::chrono::duration<double, std::milli>(now - t).count());
        t = now;
    }
};

}  // namespace

hipError_t upload_topology(DevPlan& d, const Plan& topo, const BoxDev* boxdev, hipStream_t s) {
    const int64_t nc = (int64_t)topo.cells.size(), nl = (int64_t)topo.leaf_cell.size();
    std::vector<int32_t> cell(4 * nc), aux(4 * nc), leaf(4 * nl);
    for (int64_t k = 0; k < nc; ++k) {
        const Cell& c = topo.cells[k];
        cell[4 * k] = c.first;
        cell[4 * k + 1] = c.count;
        cell[4 * k + 2] = c.parent;
        cell[4 * k + 3] = c.leaf;
        aux[4 * k] = c.child[0];
        aux[4 * k + 1] = c.child[1];
        aux[4 * k + 2] = c.box;
        aux[4 * k + 3] = c.depth;
    }
    for (int64_t l = 0; l < nl; ++l) {
        const Cell& c = topo.cells[topo.leaf_cell[l]];
        leaf[4 * l] = c.first;
        leaf[4 * l + 1] = c.count;
        leaf[4 * l + 2] = c.box;
        leaf[4 * l + 3] = topo.leaf_cell[l];
    }
    const int nbox = (int)topo.boxes.size();
    std::vector<WalkBox> wb(nbox);
    std::vector<BoxDev> bd(boxdev, boxdev + nbox);
    for (int b = 0; b < nbox; ++b) {
        const BoxParams& p = topo.boxes[b];
        const double rc2 = p.r_cut * p.r_cut;
        wb[b].L = p.box;
        wb[b].rc2_drop = rc2 * (1.0 + kGuard);
        wb[b].rc2_m2l = rc2 * (1.0 - kGuard);
        wb[b].th2 = p.theta * p.theta;
        wb[b].use_m2l = (p.order >= 0 && p.theta > 0.0) ? 1 : 0;
        wb[b].centre_cut = p.m2l_cut == 1 ? 1 : 0;
        wb[b].rc2 = rc2;
    }
    std::vector<int32_t> bfc(topo.box_first_cell.begin(), topo.box_first_cell.end());
    d.walk_levels = 0;      // a new shape: size the walk level by level once

    // Subtrees finished by k_orb_fused: the highest cells with at most fuse
    // particles and kFuseC cells (cells are in pre-order, so a subtree is the
    // contiguous id range [c, c + sub[c])).  A leaf (<= 64 particles) always
    // qualifies, so the subtrees cover every leaf; the level loop partitions
    // the cells above them, all of which split.  fuse is kFuseM where that
    // gives every CU a subtree, and down to a quarter of it below: with
    // kFuseM throughout, 32^3 particles were four workgroups of nine levels
    // at 16 us each; a quarter trades two of the loop's levels (23 us each)
    // for seven levels at 5 us (whole build, before -> after: 40^3 455 -> 397
    // us, 64^3 572 -> 536, 100^3 1071 -> 1051; 12^3 to 32^3 within the spread).
    int fuse = kFuseM;
    while (fuse > kFuseM / 4 && topo.n / 256 <= fuse / 2) fuse /= 2;
    std::vector<int32_t> sub(nc, 1), deep(nc, 0);
    for (int64_t k = nc - 1; k >= 0; --k) {
        const Cell& c = topo.cells[k];
        deep[k] = c.depth;
        if (c.child[0] >= 0) {
            sub[k] = 1 + sub[c.child[0]] + sub[c.child[1]];
            deep[k] = std::max(deep[c.child[0]], deep[c.child[1]]);
        }
    }
    auto fusable = [&](int64_t k) {
        return topo.cells[k].count <= fuse && sub[k] <= kFuseC;
    };
    std::vector<int32_t> roots, split(nc, 0), loop_cells, loop_tiles;
    std::vector<int32_t> loop_begin(1, 0);
    for (int64_t k = 0; k < nc; ++k) {
        const Cell& c = topo.cells[k];
        if (!fusable(k)) {
            if (c.child[0] < 0) return hipErrorInvalidValue;   // a leaf above kFuseM
            split[k] = 1;
        } else if (c.parent < 0 || !fusable(c.parent)) {
            roots.push_back((int32_t)k);
            roots.push_back(sub[k]);
            roots.push_back(c.depth);
            roots.push_back(deep[k]);
        }
    }
    // per level of the loop: its cells (first, count, id, left marks before
    // them; the pre-order within a depth is the position order) and each
    // tile's first cell
    const int64_t n_tiles = (topo.n + kLvTile - 1) / kLvTile;
    for (int dep = 0; dep + 1 < (int)topo.depth_begin.size(); ++dep) {
        const size_t before = loop_cells.size();
        uint32_t marks = 0;
        for (int q = topo.depth_begin[dep]; q < topo.depth_begin[dep + 1]; ++q) {
            const int32_t k = topo.cells_by_depth[q];
            if (!split[k]) continue;
            const Cell& c = topo.cells[k];
            for (int32_t v : {c.first, c.count, k, (int32_t)marks}) loop_cells.push_back(v);
            marks += (uint32_t)(c.count / 2);
        }
        if (loop_cells.size() == before) break;
        size_t at = before;
        for (int64_t b = 0; b < n_tiles; ++b) {
            while (at < loop_cells.size() && (int64_t)loop_cells[at] + loop_cells[at + 1] <= b * kLvTile) at += 4;
            loop_tiles.push_back((int32_t)((at - before) / 4));
        }
        loop_begin.push_back((int32_t)(loop_cells.size() / 4));
    }
    d.n_froots = (int)(roots.size() / 4);
    d.loop_depth_begin = loop_begin;
    hipError_t e;
    if ((e = up(d.cell, cell, s)) != hipSuccess) return e;
    if ((e = up(d.cell_aux, aux, s)) != hipSuccess) return e;
    if ((e = up(d.leaf, leaf, s)) != hipSuccess) return e;
    if ((e = up(d.level_cells, topo.cells_by_depth, s)) != hipSuccess) return e;
    if ((e = up(d.loop_cells, loop_cells, s)) != hipSuccess) return e;
    if ((e = up(d.loop_tiles, loop_tiles, s)) != hipSuccess) return e;
    if ((e = d.cell_axis.ensure(loop_cells.size() + 16)) != hipSuccess) return e;
    if ((e = up(d.froots, roots, s)) != hipSuccess) return e;
    if ((e = up(d.box_first, topo.box_first_particle, s)) != hipSuccess) return e;
    if ((e = up(d.walkbox, wb, s)) != hipSuccess) return e;
    if ((e = up(d.boxes, bd, s)) != hipSuccess) return e;
    if ((e = up(d.item_count, bfc, s)) != hipSuccess) return e;   // box -> root cell (scratch reuse)
    return hipStreamSynchronize(s);
}

std::string gpu_build_plan(DevPlan& d, const Plan& topo, const double* pos, const double* mass,
                           int chunk, hipStream_t s, PlanCounts& out, std::string* input_error,
                           const M2LReady& on_m2l, hipStream_t side) {
    input_error->clear();
    const int64_t n = topo.n;
    const int nbox = (int)topo.boxes.size();
    const int64_t nc = (int64_t)topo.cells.size(), nl = (int64_t)topo.leaf_cell.size();
    PhaseTimer clk(s);

    // ---- wrap, sort each axis by (coordinate, caller index)
    TRY(d.wpos.ensure(n * 24));
    TRY(d.keys.ensure(n * 24));
    TRY(d.plist.ensure(n * 12));
    TRY(d.plist_tmp.ensure(n * 12));
    TRY(d.keys_tmp.ensure(n * 24));
    TRY(d.wcount.ensure((kCtlAt + kCtlWords) * 4));
    TRY(d.rowcnt.ensure((nl + 2) * 4));
    TRY(d.rowcnt_m2l.ensure((nc + 2) * 4));
    TRY(d.m2l_row.ensure((nc + 1) * 4));
    hipLaunchKernelGGL(k_init, dim3(grid_of(std::max<int64_t>(nc + 2, kCtlAt + kCtlWords))), dim3(256), 0, s,
                       d.wcount.as<int32_t>(), d.rowcnt.as<int32_t>(), (int)nl + 2,
                       d.rowcnt_m2l.as<int32_t>(), (int)nc + 2, d.m2l_row.as<int32_t>(), (int)nc + 1);
    const int key_bits = n <= kKey24Max ? 24 : 32;
    hipLaunchKernelGGL(k_prepare, dim3(grid_of(n)), dim3(256), 0, s, pos, mass, n,
                       d.box_first.as<int32_t>(), nbox, d.boxes.as<BoxDev>(), d.wpos.as<double>(),
                       d.keys.as<uint32_t>(), d.plist.as<uint32_t>(), key_bits, d.wcount.as<int>());
    TRY(hipGetLastError());
    // the three axis lists are three segments of one sort: by the key,
    // then each run of equal keys by coordinate
    TRY(d.hist.ensure((size_t)sort_hist_words(n, 3) * 4));
    uint32_t* v = d.plist.as<uint32_t>();
    uint32_t* vt = d.plist_tmp.as<uint32_t>();
    bool in_tmp = false;
    if (n > 1) {
        TRY(radix_sort_u32(d.keys.as<uint32_t>(), v, d.keys_tmp.as<uint32_t>(), vt,
                           d.hist.as<uint32_t>(), n, 0, key_bits, s, &in_tmp, 3));
        if (in_tmp) {
            // the sorted keys and lists are the scratch buffers now
            std::swap(d.keys, d.keys_tmp);
            std::swap(d.plist, d.plist_tmp);
            v = d.plist.as<uint32_t>();
            vt = d.plist_tmp.as<uint32_t>();
        }
        hipLaunchKernelGGL(k_run_fix, dim3(grid_of(3 * n)), dim3(256), 0, s, d.keys.as<uint32_t>(), v,
                           n, d.wpos.as<double>(), reinterpret_cast<int*>(d.wcount.p) + 2);
        TRY(hipGetLastError());
    }
    // The input checks (wcount[0..1]) and the long-run flag (wcount[2]) come
    // back with the walk's counts, in the same round trip: with bad input
    // the tree is built on wrapped (finite) coordinates and then dropped;
    // with a long run the build is redone with the 64-bit sort (force64).
    {
        if (d.force64) {
            // coordinates closer than the key resolves, out of order
            // in a long run: sort by the full keys
            uint64_t* k = d.keys.as<uint64_t>();
            uint64_t* kt = d.keys_tmp.as<uint64_t>();
            hipLaunchKernelGGL(k_keys64, dim3(grid_of(n)), dim3(256), 0, s, d.wpos.as<double>(), n, k,
                               v);
            TRY(hipGetLastError());
            TRY(radix_sort_u64(k, v, kt, vt, d.hist.as<uint32_t>(), n, 0, 64, s, &in_tmp, 3));
            if (in_tmp) TRY(hipMemcpyAsync(v, vt, n * 12, hipMemcpyDeviceToDevice, s));
        }
    }
    if (n > 1 && nbox > 1) {
        // then stably by box: each box's particles in coordinate order
        uint32_t* k = d.keys.as<uint32_t>();
        hipLaunchKernelGGL(k_box_keys, dim3(grid_of(3 * n)), dim3(256), 0, s, v, 3 * n,
                           d.box_first.as<int32_t>(), nbox, k);
        TRY(hipGetLastError());
        TRY(radix_sort_u32(k, v, d.keys_tmp.as<uint32_t>(), vt, d.hist.as<uint32_t>(), n, 0,
                           bits_for(nbox - 1) + 1, s, &in_tmp, 3));
        if (in_tmp) TRY(hipMemcpyAsync(v, vt, n * 12, hipMemcpyDeviceToDevice, s));
    }

    clk.lap("sort");
    // ---- ORB levels
    // mark bytes at 0, then the particles' mark bits, then the lists' mark
    // words; k_orb_fused reuses the buffer for n int32
    const int64_t bits_off = (n + 255) / 256 * 256, nwords = (n + 63) / 64;
    TRY(d.flag.ensure(std::max<int64_t>(n * 4, bits_off + 4 * nwords * 8)));
    uint64_t* bits = reinterpret_cast<uint64_t*>(d.flag.as<uint8_t>() + bits_off);
    uint64_t* marks = bits + nwords;
    const bool packed = n > kLvByteMax;
    const int64_t lv_tiles = (n + kLvTile - 1) / kLvTile;
    // per-list tile sums, their scan (large n) and the scan's scratch
    TRY(d.tile_sums.ensure((6 * lv_tiles + sort_tiles(3 * lv_tiles)) * 4 + 16));
    TRY(d.clo.ensure(nc * 24));
    TRY(d.chi.ensure(nc * 24));
    // the level loop partitions the cells above the fused subtrees
    const int nloop = (int)d.loop_depth_begin.size() - 1;
    for (int dep = 0; dep < nloop; ++dep) {
        const int c0 = d.loop_depth_begin[dep], ncd = d.loop_depth_begin[dep + 1] - c0;
        const LevelCells lv{d.loop_cells.as<int4>() + c0, d.loop_tiles.as<int32_t>() + dep * lv_tiles, ncd,
                            d.cell_axis.as<int32_t>() + c0};
        hipLaunchKernelGGL(k_level_flag, dim3(lv_tiles), dim3(kLvThreads), 0, s, n, lv,
                           d.plist.as<uint32_t>(), d.wpos.as<double>(), d.clo.as<double>(),
                           d.chi.as<double>(), d.flag.as<uint8_t>(), dep + 1, dep == 0);
        if (packed)
            hipLaunchKernelGGL(k_pack_marks, dim3(grid_of(n)), dim3(256), 0, s, n,
                               d.flag.as<uint8_t>(), dep + 1, bits);
        hipLaunchKernelGGL(packed ? k_level_sums<true> : k_level_sums<false>, dim3(lv_tiles),
                           dim3(kLvThreads), 0, s, n, lv, d.plist.as<uint32_t>(),
                           d.flag.as<uint8_t>(), dep + 1, bits, marks, nwords,
                           d.tile_sums.as<uint32_t>(), (int)lv_tiles);
        TRY(hipGetLastError());
        uint32_t* offs = d.tile_sums.as<uint32_t>() + 3 * lv_tiles;
        if (lv_tiles > kLvSumMax)
            TRY(exclusive_scan_i32(d.tile_sums.as<int32_t>(), reinterpret_cast<int32_t*>(offs),
                                   3 * lv_tiles, offs + 3 * lv_tiles, s));
        hipLaunchKernelGGL(lv_tiles > kLvSumMax ? k_level_move<true> : k_level_move<false>,
                           dim3(lv_tiles), dim3(kLvThreads), 0, s, n, lv, d.plist.as<uint32_t>(),
                           d.plist_tmp.as<uint32_t>(), marks, nwords, d.tile_sums.as<uint32_t>(),
                           offs, (int)lv_tiles);
        TRY(hipGetLastError());
        std::swap(d.plist, d.plist_tmp);
    }
    // the subtrees below, each in one workgroup; leaves into perm
    TRY(d.perm.ensure(n * 4));
    hipLaunchKernelGGL(k_orb_fused, dim3(d.n_froots), dim3(kFuseT), 0, s, d.froots.as<int4>(),
                       d.cell.as<int4>(), d.cell_aux.as<int4>(), d.plist.as<uint32_t>(), n,
                       d.wpos.as<double>(), d.flag.as<int32_t>(), d.clo.as<double>(),
                       d.chi.as<double>(), d.perm.as<int32_t>());
    TRY(hipGetLastError());

    clk.lap("levels");
    // ---- leaf order, geometry, particle records
    TRY(d.leafc.ensure(nl * 32));
    TRY(d.cellc.ensure(nc * 32));
    TRY(d.wcell.ensure(nc * sizeof(WalkCell)));
    hipLaunchKernelGGL(k_geom, dim3(grid_of(nc)), dim3(256), 0, s, (int)nc, d.clo.as<double>(),
                       d.chi.as<double>(), d.cell.as<int4>(), d.cell_aux.as<int4>(),
                       d.cellc.as<double4>(), d.wcell.as<WalkCell>(), d.leafc.as<double4>());
    TRY(hipGetLastError());
    TRY(d.x64.ensure(n * 32 + kReadAhead));
    TRY(d.x32.ensure(n * 16 + kReadAhead));
    GatherArgs g{pos, mass, d.perm.as<int32_t>(), d.leaf.as<int4>(), d.leafc.as<double4>(),
                 d.boxes.as<BoxDev>(), d.x64.as<double4>(), d.x32.as<float4>(), (int32_t)nl};
    // With a side stream the particle records are gathered there, beside the
    // walk (which reads only the cells); s waits for them before the build
    // returns (and before any early return).
    const bool side_gather = side != nullptr && side != s;
    if (side_gather) {
        for (hipEvent_t* e : {&d.geom_ev, &d.gather_ev})
            if (!*e) TRY(hipEventCreateWithFlags(e, hipEventDisableTiming));
        TRY(hipEventRecord(d.geom_ev, s));
        TRY(hipStreamWaitEvent(side, d.geom_ev, 0));
        TRY(launch_gather(g, nullptr, side));
        TRY(hipEventRecord(d.gather_ev, side));
    } else {
        TRY(launch_gather(g, nullptr, s));
    }
    auto join_gather = [&]() -> hipError_t {
        return side_gather ? hipStreamWaitEvent(s, d.gather_ev, 0) : hipSuccess;
    };

    clk.lap("records");
    // ---- dual walk
    // the canonical half of (root, root, s): the zero shift and the 13
    // shifts with code > 13
    const int64_t nf0 = 14 * (int64_t)nbox;
    std::vector<int32_t> f0(2 * nf0);
    for (int b = 0; b < nbox; ++b)
        for (int q = 0; q < 14; ++q) {
            const int root = topo.box_first_cell[b];
            f0[2 * (14 * b + q)] = root;
            f0[2 * (14 * b + q) + 1] = (root << 5) | (13 + q);
        }
    int64_t n_p2p = 0, n_m2l = 0;
    int32_t dmin_src = 0x7fffffff, dmin_tgt = 0x7fffffff;
    bool done = false;
    bool any_m2l = false;
    for (const BoxParams& b : topo.boxes) any_m2l = any_m2l || (b.order >= 0 && b.theta > 0.0);
    int flags[3] = {0, 0, 0};
    bool have_flags = false;
    const int2 ks = make_int2(5 + bits_for((uint64_t)std::max<int64_t>(1, nl - 1)),
                              5 + bits_for((uint64_t)std::max<int64_t>(1, nc - 1)));
    // Level-by-level walk without host round trips, sized from the previous
    // build of the same tree shape; falls back to the host-driven loop.
    if (d.walk_cap_front > 0 && d.walk_levels > 0 && d.walk_levels + 16 <= kCtlWords) {
        const uint32_t capf = d.walk_cap_front, capp = d.walk_cap_p2p, capm = d.walk_cap_m2l;
        const int L = d.walk_levels;
        TRY(d.front.ensure((size_t)std::max<int64_t>(capf, nf0) * 8));
        TRY(d.front_next.ensure((size_t)capf * 8));
        TRY(d.p2p_keys.ensure((size_t)capp * 8));
        TRY(d.m2l_keys.ensure((size_t)std::max<uint32_t>(capm, 1) * 8));
        DevBuf* bufs[2] = {&d.front, &d.front_next};
        // the top levels in one workgroup while the last build's frontiers
        // were small (any size is handled; this only chooses the split),
        // then two levels per launch up to level Le >= L
        int top = 0;
        while (top < L && top < (int)d.walk_sizes.size() && d.walk_sizes[top] <= kWalkTopMax) ++top;
        const int Le = top + 2 * ((L - top + 1) / 2);
        uint32_t* ctl = d.wcount.as<uint32_t>() + kCtlAt;   // cleared by k_init
        uint32_t* sizes = ctl + 4;
        hipLaunchKernelGGL(k_walk_top, dim3(1), dim3(kWalkT), 0, s, nbox, d.item_count.as<int32_t>(),
                           d.front.as<int2>(), d.front_next.as<int2>(), top, sizes, ctl, capf,
                           capp, capm, d.walkbox.as<WalkBox>(), d.wcell.as<WalkCell>(), ks,
                           d.p2p_keys.as<uint64_t>(), d.m2l_keys.as<uint64_t>());
        int cur = walk_top_steps(top) & 1;   // the buffer that holds level `top`
        for (int it = top; it < L; it += 2) {
            // workgroups for the frontier the last build had at this level
            // (the kernel strides over any size; this only trims launches)
            const int64_t prev = it < (int)d.walk_sizes.size() ? d.walk_sizes[it] : capf;
            const bool narrow = prev <= kWalkNarrowMax;
            const int T = narrow ? kWalkNarrow : kWalkT;
            const unsigned g = (unsigned)std::min<int64_t>(kWalkThreads / T, (prev + prev / 4 + 2 * T) / T);
            hipLaunchKernelGGL(narrow ? k_walk_multi<kWalkNarrow> : k_walk_multi<kWalkT>, dim3(g), dim3(T),
                               0, s, bufs[cur]->as<int2>(),
                               bufs[cur ^ 1]->as<int2>(), it, sizes, ctl, capf, capp, capm,
                               d.walkbox.as<WalkBox>(), d.wcell.as<WalkCell>(), ks,
                               d.p2p_keys.as<uint64_t>(), d.m2l_keys.as<uint64_t>());
            cur ^= 1;
        }
        if (any_m2l)
            hipLaunchKernelGGL(k_m2l_depths, dim3(8), dim3(256), 0, s, d.m2l_keys.as<uint64_t>(),
                               ctl + 1, capm, ks.y, d.cell_aux.as<int4>(), ctl + 5 + Le);
        TRY(hipGetLastError());
        // the walk's counts and the input checks in one round trip, into
        // pinned memory
        TRY(d.ensure_host_rb());
        TRY(hipMemcpyAsync(d.host_rb, d.wcount.p, (kCtlAt + Le + 7) * 4, hipMemcpyDeviceToHost, s));
        TRY(hipStreamSynchronize(s));
        std::vector<uint32_t> hc(d.host_rb + kCtlAt, d.host_rb + kCtlAt + Le + 7);
        std::memcpy(flags, d.host_rb, 12);
        have_flags = true;
        if (clk.on) {
            std::fprintf(stderr, "[pmfmm gpu plan] walk frontier per level:");
            for (int it = 0; it <= Le; ++it) std::fprintf(stderr, " %u", hc[4 + it]);
            std::fprintf(stderr, "\n");
        }
        if (hc[2] == 0 && hc[4 + Le] == 0 && hc[0] <= capp && hc[1] <= capm) {
            n_p2p = hc[0];
            n_m2l = hc[1];
            dmin_tgt = (int32_t)(0x7fffffffu - hc[5 + Le]);
            dmin_src = (int32_t)(0x7fffffffu - hc[6 + Le]);
            d.walk_sizes.assign(hc.begin() + 4, hc.begin() + 4 + L);
            done = true;
        }
    }
    if (!done) {
        int64_t nf = nf0;
        TRY(d.front.ensure(std::max<size_t>(f0.size() * 4, 4096)));
        TRY(hipMemcpyAsync(d.front.p, f0.data(), f0.size() * 4, hipMemcpyHostToDevice, s));
        // this loop's counters: wcount[20..23] (words 0..2 hold the checks)
        uint32_t* wc = d.wcount.as<uint32_t>() + 20;
        hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, wc, 4);
        // (an overflowed walk above has left its keys' counts elsewhere)
        if (d.p2p_keys.bytes < 16) TRY(d.p2p_keys.ensure(1 << 20));
        if (d.m2l_keys.bytes < 16) TRY(d.m2l_keys.ensure(1 << 16));
        uint32_t hc[4] = {0, 0, 0, 0};
        int levels = 0;
        int64_t max_front = nf;
        d.walk_sizes.clear();
        while (nf > 0) {
            d.walk_sizes.push_back((uint32_t)nf);
            TRY(d.front_next.grow((size_t)4 * nf * 8, 0, s));
            // each pair adds at most 4 children and 2 keys (itself and mirror)
            if ((size_t)(n_p2p + 2 * nf) * 8 > d.p2p_keys.bytes)
                TRY(d.p2p_keys.grow((size_t)(n_p2p + 2 * nf) * 8 * 2, (size_t)n_p2p * 8, s));
            if ((size_t)(n_m2l + 2 * nf) * 8 > d.m2l_keys.bytes)
                TRY(d.m2l_keys.grow((size_t)(n_m2l + 2 * nf) * 8 * 2, (size_t)n_m2l * 8, s));
            hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, wc, 1);
            hipLaunchKernelGGL(k_walk, dim3(grid_of(nf)), dim3(256), 0, s, d.front.as<int2>(), (int)nf,
                               d.front_next.as<int2>(), d.walkbox.as<WalkBox>(), d.wcell.as<WalkCell>(),
                               ks, wc, d.p2p_keys.as<uint64_t>(), d.m2l_keys.as<uint64_t>());
            TRY(hipGetLastError());
            TRY(hipMemcpyAsync(hc, wc, 16, hipMemcpyDeviceToHost, s));
            TRY(hipStreamSynchronize(s));
            nf = hc[0];
            n_p2p = hc[1];
            n_m2l = hc[2];
            max_front = std::max<int64_t>(max_front, nf);
            ++levels;
            std::swap(d.front, d.front_next);
        }
        if (n_m2l > 0) {
            // smallest M2L depths (words 4, 5 of wcount, zeroed here)
            uint32_t cnt32 = (uint32_t)n_m2l;
            TRY(hipMemcpyAsync(d.wcount.as<uint32_t>() + 6, &cnt32, 4, hipMemcpyHostToDevice, s));
            hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, d.wcount.as<uint32_t>() + 4, 2);
            hipLaunchKernelGGL(k_m2l_depths, dim3(8), dim3(256), 0, s, d.m2l_keys.as<uint64_t>(),
                               d.wcount.as<uint32_t>() + 6, (uint32_t)n_m2l, ks.y,
                               d.cell_aux.as<int4>(), d.wcount.as<uint32_t>() + 4);
            TRY(hipGetLastError());
            uint32_t dd[2] = {0u, 0u};
            TRY(hipMemcpyAsync(dd, d.wcount.as<uint32_t>() + 4, 8, hipMemcpyDeviceToHost, s));
            TRY(hipStreamSynchronize(s));
            dmin_tgt = (int32_t)(0x7fffffffu - dd[0]);
            dmin_src = (int32_t)(0x7fffffffu - dd[1]);
        }
        // sizes for the next build of this shape (with some room to move)
        d.walk_levels = levels + 2;
        d.walk_cap_front = (uint32_t)std::min<int64_t>(0x7fffffff, max_front + max_front / 2 + 4096);
        d.walk_cap_p2p = (uint32_t)std::min<int64_t>(0x7fffffff, n_p2p + n_p2p / 4 + 4096);
        d.walk_cap_m2l = (uint32_t)std::min<int64_t>(0x7fffffff, n_m2l + n_m2l / 4 + 4096);
    }

    if (!have_flags) {
        TRY(hipMemcpyAsync(flags, d.wcount.p, 12, hipMemcpyDeviceToHost, s));
        TRY(hipStreamSynchronize(s));
    }
    if (flags[0] != 0x7fffffff || flags[1] != 0x7fffffff || (flags[2] != 0 && !d.force64))
        TRY(join_gather());
    if (flags[0] != 0x7fffffff) {
        *input_error = "non-finite position at particle " + std::to_string(flags[0]);
        return std::string();
    }
    if (flags[1] != 0x7fffffff) {
        *input_error = "negative or non-finite mass at particle " + std::to_string(flags[1]);
        return std::string();
    }
    if (flags[2] != 0 && !d.force64) {
        // a run of equal keys too long for k_run_fix: build again
        // with the full 64-bit sort
        d.force64 = true;
        std::string e = gpu_build_plan(d, topo, pos, mass, chunk, s, out, input_error, on_m2l, side);
        d.force64 = false;
        return e;
    }
    clk.lap("walk");
    // ---- canonical order and CSR
    TRY(d.p2p_row.ensure((nl + 1) * 4));
    TRY(d.js.ensure(std::max<int64_t>(1, n_p2p) * 4));
    TRY(d.m2l_src.ensure(std::max<int64_t>(1, n_m2l) * 4));
    TRY(d.m2l_shift.ensure(std::max<int64_t>(1, n_m2l) * 4));
    TRY(d.m2l_vals.ensure(std::max<int64_t>(1, n_m2l) * 4));
    // slots, then long-row scratch: two int32 per key
    TRY(d.p2p_keys_tmp.ensure(std::max<int64_t>(1, n_p2p) * 8));
    TRY(d.m2l_keys_tmp.ensure(std::max<int64_t>(1, n_m2l) * 8));
    TRY(d.longrows.ensure((nl + 1) * 4));
    TRY(d.tile_sums.ensure(sort_tiles(nl + 1) * 4 + 16));
    TRY(d.longrows_m2l.ensure((nc + 1) * 4));
    TRY(d.tile_sums_m2l.ensure(sort_tiles(nc + 1) * 4 + 16));
    struct RowList {
        const DevBuf& keys;
        int64_t nk;
        int nrows;
        int ks;
        DevBuf& row;
        DevBuf& vals;
        DevBuf& tmp;       // per-key slots, then long-row scratch
        DevBuf& cnt;       // nrows + 2 counts, cleared by k_init
        DevBuf& longs;     // nrows + 1
        DevBuf& tsums;     // scan scratch
    };
    const RowList p2p_rows{d.p2p_keys, n_p2p, (int)nl, ks.x, d.p2p_row, d.js,
                           d.p2p_keys_tmp, d.rowcnt, d.longrows, d.tile_sums};
    const RowList m2l_rows{d.m2l_keys, n_m2l, (int)nc, ks.y, d.m2l_row, d.m2l_vals,
                           d.m2l_keys_tmp, d.rowcnt_m2l, d.longrows_m2l, d.tile_sums_m2l};
    // the rows in two parts: the atomic row counts, then the rest
    auto count_rows = [&](const RowList& rl, hipStream_t st) -> hipError_t {
        if (rl.nk > 0)
            hipLaunchKernelGGL(k_row_count, dim3(grid_of(rl.nk, kRcKeys)), dim3(kRcThreads), 0, st,
                               rl.keys.as<uint64_t>(), rl.nk, rl.ks, rl.cnt.as<int32_t>(),
                               rl.tmp.as<int32_t>());
        return hipGetLastError();
    };
    auto finish_rows = [&](const RowList& rl, hipStream_t st) -> hipError_t {
        int32_t* cnt = rl.cnt.as<int32_t>();
        int32_t* slot = rl.tmp.as<int32_t>();
        hipError_t e = exclusive_scan_i32(cnt, rl.row.as<int32_t>(), rl.nrows + 1,
                                          rl.tsums.as<uint32_t>(), st);
        if (e != hipSuccess) return e;
        if (rl.nk > 0) {
            hipLaunchKernelGGL(k_row_place, dim3(grid_of(rl.nk)), dim3(256), 0, st,
                               rl.keys.as<uint64_t>(), rl.nk, rl.ks, rl.row.as<int32_t>(), slot,
                               rl.vals.as<int32_t>());
            // the count of long rows goes in cnt[nrows + 1] (zeroed above)
            int32_t* nlong = cnt + rl.nrows + 1;
            hipLaunchKernelGGL(k_row_sort_short, dim3((rl.nrows + 3) / 4), dim3(256), 0, st,
                               rl.row.as<int32_t>(), rl.nrows, rl.vals.as<int32_t>(),
                               rl.longs.as<int32_t>(), nlong);
            hipLaunchKernelGGL(k_row_sort_long, dim3(64), dim3(256), 0, st, rl.row.as<int32_t>(),
                               rl.vals.as<int32_t>(), rl.longs.as<int32_t>(), nlong, slot,
                               row_lds_cap());
        }
        return hipGetLastError();
    };
    // With M2L tasks and a side stream, the M2L rows and then the far field
    // (on_m2l) run on the side stream while the P2P rows and the work items
    // are built on s; the side stream starts after everything before it on
    // s (the walk), and s waits for the M2L rows (not the far field) before
    // the build ends.
    const bool fork = side != nullptr && side != s && n_m2l > 0;
    hipStream_t ms = s;
    if (fork) {
        for (hipEvent_t* e : {&d.fork_ev, &d.m2l_done})
            if (!*e) TRY(hipEventCreateWithFlags(e, hipEventDisableTiming));
        TRY(hipEventRecord(d.fork_ev, s));
        TRY(hipStreamWaitEvent(side, d.fork_ev, 0));
        ms = side;
        // the P2P row counts (a long kernel) first, so the device has work
        // on s while the host enqueues the side stream's launches
        TRY(count_rows(p2p_rows, s));
    }
    // M2L rows (all empty, as k_init left them, without tasks), sources and
    // shifts; the smallest depths go to wcount words 16, 17 (the walk's
    // k_m2l_depths gave the same values to the host already)
    if (n_m2l > 0) {
        TRY(count_rows(m2l_rows, ms));
        TRY(finish_rows(m2l_rows, ms));
        hipLaunchKernelGGL(k_m2l_split, dim3(grid_of(nc)), dim3(256), 0, ms, d.m2l_row.as<int32_t>(),
                           (int)nc, d.m2l_vals.as<int32_t>(), d.cell_aux.as<int4>(),
                           d.m2l_src.as<int32_t>(), d.m2l_shift.as<int32_t>(),
                           reinterpret_cast<int32_t*>(d.wcount.p) + 16);
    }
    TRY(hipGetLastError());
    if (fork) TRY(hipEventRecord(d.m2l_done, side));
    if (!fork) TRY(count_rows(p2p_rows, s));
    if (on_m2l) {
        std::string e = on_m2l(n_m2l, dmin_src, dmin_tgt);
        if (!e.empty()) return e;
    }
    TRY(finish_rows(p2p_rows, s));
    if (fork) TRY(hipStreamWaitEvent(s, d.m2l_done, 0));
    TRY(join_gather());
    out.n_p2p = n_p2p;
    out.n_m2l = n_m2l;
    clk.lap("csr");
    std::string e2 = gpu_make_items(d, topo, n_p2p, chunk, s, out);
    clk.lap("items");
    return e2;
}

std::string gpu_make_items(DevPlan& d, const Plan& topo, int64_t n_p2p, int chunk, hipStream_t s,
                           PlanCounts& out) {
    const int64_t nl = (int64_t)topo.leaf_cell.size();
    if (chunk <= 0) chunk = auto_chunk(n_p2p, nl);
    TRY(d.cost.ensure((nl + 1) * 4));
    TRY(d.leaf_slot.ensure((nl + 1) * 4));
    TRY(d.tile_sums.ensure(sort_tiles(nl + 1) * 4 + 16));
    TRY(d.wcount.ensure((kCtlAt + kCtlWords) * 4));
    hipLaunchKernelGGL(k_item_count, dim3(grid_of(nl + 1)), dim3(256), 0, s, (int)nl,
                       d.p2p_row.as<int32_t>(), chunk, d.cost.as<int32_t>(), d.wcount.as<uint32_t>());
    TRY(hipGetLastError());
    TRY(exclusive_scan_i32(d.cost.as<int32_t>(), d.leaf_slot.as<int32_t>(), nl + 1,
                           d.tile_sums.as<uint32_t>(), s));
    // buffers sized for the most items the rows can give (sum over rows of
    // ceil(len / chunk) <= n_p2p / chunk + rows), so the count is read back
    // only at the end
    const int64_t cap = std::max<int64_t>(1, (n_p2p + chunk - 1) / chunk + nl);
    TRY(d.items.ensure(cap * 16));
    TRY(d.item_cost.ensure(cap));
    TRY(d.rowcand.ensure(nl * 8));
    TRY(d.queue.ensure(cap * 4));
    // largest item: chunk tasks of at most 64 x 64 pairs
    const int cshift = std::max(0, bits_for((uint64_t)chunk * 64 * 64) - 8);
    hipLaunchKernelGGL(k_items, dim3(grid_of(nl * 64)), dim3(256), 0, s, (int)nl,
                       d.p2p_row.as<int32_t>(), d.js.as<int32_t>(), d.leaf.as<int4>(), chunk, cshift,
                       d.leaf_slot.as<int32_t>(), d.items.as<int4>(), d.item_cost.as<uint8_t>(),
                       d.rowcand.as<unsigned long long>());
    hipLaunchKernelGGL(k_queue, dim3(kQueueSegs), dim3(1024), 0, s, (int)nl, d.leaf_slot.as<int32_t>(),
                       d.item_cost.as<uint8_t>(), d.rowcand.as<unsigned long long>(),
                       d.queue.as<uint32_t>(), d.wcount.as<uint32_t>());
    TRY(hipGetLastError());
    // words 8, 9: candidate pairs; 10: items; 16, 17: M2L depths (set by the build)
    uint32_t w[10];
    TRY(d.ensure_host_rb());
    TRY(hipMemcpyAsync(d.host_rb, d.wcount.as<uint32_t>() + 8, sizeof(w), hipMemcpyDeviceToHost, s));
    TRY(hipStreamSynchronize(s));
    std::memcpy(w, d.host_rb, sizeof(w));
    unsigned long long cand = 0;
    std::memcpy(&cand, w, 8);
    const int64_t n_items = (int64_t)w[2];
    TRY(d.partial.ensure(std::max<int64_t>(1, n_items) * 4 * 64 * 8));
    out.n_items = n_items;
    out.candidate_pairs = (int64_t)cand;
    out.m2l_min_depth_src = (int32_t)w[8];
    out.m2l_min_depth_tgt = (int32_t)w[9];
    return std::string();
}

}  // namespace pmfmm
