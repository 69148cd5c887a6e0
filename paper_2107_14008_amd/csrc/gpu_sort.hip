// Device primitives of the on-GPU planner: a stable LSD radix sort of 64-bit
// or 32-bit keys (optionally carrying 32-bit values), also of several
// equal-length segments at once, and an exclusive prefix sum of 32-bit
// integers.
//
// Radix sort: 8-bit digits, tiles of 4096 elements (256 threads x 16
// rounds; 1024 for segments under kSmallSortN elements, whose few tiles
// would otherwise leave most CUs idle); a tile never straddles two segments.
// Per pass: (1) per-tile digit histogram in LDS, stored [segment][digit][tile];
// (2) an exclusive scan of each row of tiles, one workgroup per row, and the
// row's total; (3) scatter: the 256 row totals of the segment, scanned by
// each workgroup, give the digits' starts; inside a tile each wavefront takes
// 64 R consecutive elements, loaded at once, and ranks them 64 at a time per
// digit with ballots (eight ballots give each lane the mask of lanes holding
// its digit) and a running per-digit count of its own in LDS, so the order of
// equal digits is kept (stable), which makes the sort stable across passes;
// the tile is ordered in LDS and written out in runs.  With the four
// wavefronts sharing each round's 256 elements, a round was three barriers and
// a load behind them: a scatter of 3 x 128^3 pairs 46 us, now 36; 3 x 256^3
// 368, now 261 (the reads and writes alone 175).  Up to kDirectTiles tiles per segment the scatter adds up its row of
// the histogram itself and (2) is left out (12 us less per build at 4,096
// particles; at 262,144, 256 tiles, its serial sums would cost more than the
// launch).
#include <algorithm>

#include "gpu_plan.h"

namespace pmfmm {
namespace {

constexpr int kThreads = 256;
constexpr int kRounds = 16;
constexpr int kTile = kThreads * kRounds;  // 4096
constexpr int kRoundsSmall = 4;
constexpr int64_t kSmallSortN = int64_t(1) << 20;

int radix_rounds(int64_t n) { return n < kSmallSortN ? kRoundsSmall : kRounds; }

int64_t radix_tiles(int64_t n) {
    const int64_t t = (int64_t)kThreads * radix_rounds(n);
    return (n + t - 1) / t;
}

// Block b handles tile (b % tiles) of segment (b / tiles); its elements are
// [seg n + tile T, min(seg n + (tile + 1) T, (seg + 1) n)), T = 256 R.
struct TileRange {
    int64_t begin, end;
    size_t col;   // (seg * 256) * tiles + tile: add digit * tiles
};

template <int R>
__device__ __forceinline__ TileRange tile_range(int64_t n, int tiles) {
    const int seg = blockIdx.x / tiles, tile = blockIdx.x - seg * tiles;
    TileRange t;
    t.begin = (int64_t)seg * n + (int64_t)tile * (kThreads * R);
    t.end = min((int64_t)seg * n + n, t.begin + kThreads * R);
    t.col = (size_t)seg * 256 * tiles + tile;
    return t;
}

template <class K, int R>
__global__ void __launch_bounds__(kThreads)
rs_hist(const K* __restrict__ keys, int64_t n, int shift, uint32_t* __restrict__ hist,
        int tiles) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const TileRange tr = tile_range<R>(n, tiles);
    K k[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = tr.begin + r * kThreads + threadIdx.x;
        k[r] = i < tr.end ? keys[i] : K(0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = tr.begin + r * kThreads + threadIdx.x;
        if (i < tr.end) atomicAdd(&h[(k[r] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[tr.col + (size_t)threadIdx.x * tiles] = h[threadIdx.x];
}

constexpr int kDirectTiles = 32;

// Exclusive scan of one row of `tiles` counts (in place) and its total, one
// workgroup per [segment][digit] row.
__global__ void __launch_bounds__(kThreads)
rs_rowscan(uint32_t* __restrict__ hist, int tiles, uint32_t* __restrict__ total) {
    __shared__ uint32_t wsum[kThreads / 64];
    uint32_t* __restrict__ row = hist + (size_t)blockIdx.x * tiles;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t carry = 0;
    for (int b = 0; b < tiles; b += kThreads) {
        const int k = b + t;
        const uint32_t v = k < tiles ? row[k] : 0u;
        uint32_t x = v;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        if (lane == 63) wsum[wave] = x;
        __syncthreads();
        uint32_t before = carry, all = 0;
        for (int w = 0; w < kThreads / 64; ++w) {
            if (w < wave) before += wsum[w];
            all += wsum[w];
        }
        if (k < tiles) row[k] = before + x - v;
        carry += all;
        __syncthreads();
    }
    if (t == 0) total[blockIdx.x] = carry;
}

// Exclusive scan of m 32-bit values by one workgroup of 1024 threads.
__global__ void __launch_bounds__(1024) scan_single(uint32_t* __restrict__ a, int64_t m) {
    __shared__ uint32_t part[1024];
    const int t = threadIdx.x;
    const int64_t per = (m + 1023) / 1024;
    const int64_t b = t * per, e = min(m, b + per);
    uint32_t s = 0;
    for (int64_t i = b; i < e; ++i) s += a[i];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < 1024; off <<= 1) {
        uint32_t v = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    uint32_t run = t == 0 ? 0u : part[t - 1];
    for (int64_t i = b; i < e; ++i) {
        const uint32_t v = a[i];
        a[i] = run;
        run += v;
    }
}

// Scatter of one pass.  The tile is first put in digit order in LDS (local
// position = the digit's start in the tile + the element's stable rank among
// the tile's elements of that digit), then written out position by
// position: consecutive positions of one digit go to consecutive addresses,
// so the global writes come in runs instead of one element per line.
//
// DIRECT: hist holds the tiles' counts; otherwise their exclusive scan by row
// (rs_rowscan), the tile's own counts being the difference to the next
// entry, and `total` the rows' totals.
template <class K, bool VALS, int R, bool DIRECT>
__global__ void __launch_bounds__(kThreads)
rs_scatter(const K* __restrict__ kin, const uint32_t* __restrict__ vin,
           K* __restrict__ kout, uint32_t* __restrict__ vout, int64_t n, int shift,
           const uint32_t* __restrict__ hist, const uint32_t* __restrict__ total, int tiles) {
    __shared__ K ks[kThreads * R];
    __shared__ uint32_t vs[VALS ? kThreads * R : 1];
    __shared__ uint32_t start[256];     // digit start inside the tile
    __shared__ uint32_t goff[256];      // digit start in the output
    __shared__ uint32_t wc[kThreads / 64][256];   // per wave: elements of each digit
    const int t = threadIdx.x;
    const int lane = t & 63, wave = t >> 6;
    const TileRange tr = tile_range<R>(n, tiles);
    const int64_t w0 = tr.begin + (int64_t)wave * (64 * R) + lane;
    K key[R];
    uint32_t val[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t i = w0 + 64 * r;
        key[r] = i < tr.end ? kin[i] : K(0);
        if (VALS) val[r] = i < tr.end ? vin[i] : 0u;
    }
    // exclusive scans over the digits of the tile's counts (start) and of the
    // segment's (one wave scans 4 digits per lane); goff: the digit's total in
    // the segment first, its start in the output for this tile in the end
    uint32_t mine;   // elements of digit t in the segment's tiles before this one
    {
        const int seg = blockIdx.x / tiles, tile = blockIdx.x - seg * tiles;
        const uint32_t* __restrict__ row = hist + ((size_t)seg * 256 + t) * tiles;
        uint32_t c, all;
        if constexpr (DIRECT) {
            mine = 0;
            all = 0;
            for (int k = 0; k < tiles; ++k) {
                const uint32_t v = row[k];
                if (k < tile) mine += v;
                all += v;
            }
            c = row[tile];
        } else {
            mine = row[tile];
            all = total[seg * 256 + t];
            c = (tile + 1 < tiles ? row[tile + 1] : all) - mine;
        }
        start[t] = c;
        goff[t] = all;
        for (int w = 0; w < kThreads / 64; ++w) wc[w][t] = 0;
    }
    __syncthreads();
    if (wave < 2) {
        uint32_t* __restrict__ a = wave == 0 ? start : goff;
        uint32_t v[4], tot = 0;
        for (int j = 0; j < 4; ++j) {
            v[j] = a[4 * lane + j];
            tot += v[j];
        }
        uint32_t x = tot;
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t y = __shfl_up(x, off);
            if (lane >= off) x += y;
        }
        uint32_t e = x - tot;
        for (int j = 0; j < 4; ++j) {
            a[4 * lane + j] = e;
            e += v[j];
        }
    }
    __syncthreads();
    goff[t] += mine + (uint32_t)((int64_t)(blockIdx.x / tiles) * n);
    // the ranks among the wave's elements of the same digit
    const uint64_t below = (1ull << lane) - 1;
    uint32_t rank[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool valid = w0 + 64 * r < tr.end;
        const uint32_t d = (uint32_t)(key[r] >> shift) & 255u;
        uint64_t m = __ballot(valid);
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t bb = __ballot(bit);
            m &= bit ? bb : ~bb;
        }
        const uint32_t first = (uint32_t)__popcll(m & below), had = wc[wave][d];
        rank[r] = had + first;
        // every lane has read the count before the first of them adds to it
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (valid && first == 0) wc[wave][d] = had + (uint32_t)__popcll(m);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    {   // each wave's start of digit t in the tile
        uint32_t at = start[t];
        for (int w = 0; w < kThreads / 64; ++w) {
            const uint32_t c = wc[w][t];
            wc[w][t] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (w0 + 64 * r >= tr.end) continue;
        const uint32_t pos = wc[wave][(uint32_t)(key[r] >> shift) & 255u] + rank[r];
        ks[pos] = key[r];
        if (VALS) vs[pos] = val[r];
    }
    __syncthreads();
    const int len = (int)(tr.end - tr.begin);
    for (int p = t; p < len; p += kThreads) {
        const K k = ks[p];
        const uint32_t d = (uint32_t)(k >> shift) & 255u;
        const uint32_t o = goff[d] + (uint32_t)p - start[d];
        kout[o] = k;
        if (VALS) vout[o] = vs[p];
    }
}

// ---- exclusive scan of int32 (tiles of 4096)
__global__ void __launch_bounds__(kThreads)
scan_tile_sums(const int32_t* __restrict__ in, int64_t n, uint32_t* __restrict__ sums) {
    __shared__ int32_t red[kThreads];
    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)threadIdx.x * kRounds;
    int32_t s = 0;
    for (int r = 0; r < kRounds; ++r)
        if (base + r < n) s += in[base + r];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = kThreads / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = (uint32_t)red[0];
}

// sums holds each tile's offset (kScanned: scan_single ran) or the tile sums
// themselves, and each workgroup adds up those before its tile (kTileSums, one
// launch fewer; for up to kApplySumMax tiles).
constexpr int kApplySumMax = 4096;

//
// KIND: kScanned; kTileSums; or kOwnSums, where each workgroup adds up the
// input before its tile itself (no scan_tile_sums launch; for up to
// kOwnSumMax elements).
enum { kScanned, kTileSums, kOwnSums };
constexpr int64_t kOwnSumMax = 32768;

template <int KIND>
__global__ void __launch_bounds__(kThreads)
scan_tile_apply(const int32_t* __restrict__ in, int32_t* __restrict__ out, int64_t n,
                const uint32_t* __restrict__ sums) {
    __shared__ int32_t part[kThreads];
    __shared__ uint32_t toff;
    const int t = threadIdx.x;
    if (KIND != kScanned) {
        uint32_t c = 0;
        if (KIND == kTileSums) {
            for (int k = t; k < (int)blockIdx.x; k += kThreads) c += sums[k];
        } else {
#pragma unroll 4
            for (int k = t; k < (int)blockIdx.x * kTile; k += kThreads) c += (uint32_t)in[k];
        }
        for (int off = 32; off > 0; off >>= 1) c += __shfl_down(c, off);
        if ((t & 63) == 0) part[t >> 6] = (int32_t)c;
        __syncthreads();
        if (t == 0) {
            uint32_t a = 0;
            for (int w = 0; w < kThreads / 64; ++w) a += (uint32_t)part[w];
            toff = a;
        }
        __syncthreads();
    }
    const int64_t base = (int64_t)blockIdx.x * kTile + (int64_t)t * kRounds;
    int32_t v[kRounds];
    int32_t s = 0;
    for (int r = 0; r < kRounds; ++r) {
        v[r] = base + r < n ? in[base + r] : 0;
        s += v[r];
    }
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < kThreads; off <<= 1) {
        int32_t x = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += x;
        __syncthreads();
    }
    int32_t run = (int32_t)(KIND == kScanned ? sums[blockIdx.x] : toff) + (t == 0 ? 0 : part[t - 1]);
    for (int r = 0; r < kRounds; ++r) {
        if (base + r < n) out[base + r] = run;
        run += v[r];
    }
}

}  // namespace

hipError_t exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, uint32_t* tile_sums,
                              hipStream_t s);

int64_t sort_tiles(int64_t n) { return (n + kTile - 1) / kTile; }

int64_t sort_hist_words(int64_t n, int nseg) {
    const int64_t m = (int64_t)nseg * 256 * radix_tiles(n);
    return m + (int64_t)nseg * 256 + 16;
}

template <class K, int R>
hipError_t radix_sort_r(K* keys, uint32_t* vals, K* tmp_keys, uint32_t* tmp_vals, uint32_t* hist,
                        int64_t n, int bit_begin, int bit_end, hipStream_t s, bool* result_in_tmp,
                        int nseg) {
    const int tiles = (int)radix_tiles(n);
    const int blocks = nseg * tiles;
    K* ka = keys;
    K* kb = tmp_keys;
    uint32_t* va = vals;
    uint32_t* vb = tmp_vals;
    // scratch layout: counts [m], then the row totals
    const int64_t m = (int64_t)nseg * 256 * tiles;
    uint32_t* total = hist + m;
    const bool direct = tiles <= kDirectTiles;
    const auto scatter = vals ? (direct ? rs_scatter<K, true, R, true> : rs_scatter<K, true, R, false>)
                              : (direct ? rs_scatter<K, false, R, true> : rs_scatter<K, false, R, false>);
    for (int shift = bit_begin; shift < bit_end; shift += 8) {
        hipLaunchKernelGGL((rs_hist<K, R>), dim3(blocks), dim3(kThreads), 0, s, ka, n, shift, hist,
                           tiles);
        if (!direct)
            hipLaunchKernelGGL(rs_rowscan, dim3(nseg * 256), dim3(kThreads), 0, s, hist, tiles, total);
        hipLaunchKernelGGL(scatter, dim3(blocks), dim3(kThreads), 0, s, ka, va, kb, vb, n, shift, hist,
                           total, tiles);
        std::swap(ka, kb);
        std::swap(va, vb);
        *result_in_tmp = !*result_in_tmp;
    }
    return hipGetLastError();
}

template <class K>
hipError_t radix_sort(K* keys, uint32_t* vals, K* tmp_keys, uint32_t* tmp_vals, uint32_t* hist,
                      int64_t n, int bit_begin, int bit_end, hipStream_t s, bool* result_in_tmp,
                      int nseg) {
    *result_in_tmp = false;
    if (n <= 1 || nseg < 1) return hipSuccess;
    if (radix_rounds(n) == kRoundsSmall)
        return radix_sort_r<K, kRoundsSmall>(keys, vals, tmp_keys, tmp_vals, hist, n, bit_begin,
                                             bit_end, s, result_in_tmp, nseg);
    return radix_sort_r<K, kRounds>(keys, vals, tmp_keys, tmp_vals, hist, n, bit_begin, bit_end, s,
                                    result_in_tmp, nseg);
}

hipError_t radix_sort_u64(uint64_t* keys, uint32_t* vals, uint64_t* tmp_keys, uint32_t* tmp_vals,
                          uint32_t* hist, int64_t n, int bit_begin, int bit_end, hipStream_t s,
                          bool* result_in_tmp, int nseg) {
    return radix_sort<uint64_t>(keys, vals, tmp_keys, tmp_vals, hist, n, bit_begin, bit_end, s,
                                result_in_tmp, nseg);
}

hipError_t radix_sort_u32(uint32_t* keys, uint32_t* vals, uint32_t* tmp_keys, uint32_t* tmp_vals,
                          uint32_t* hist, int64_t n, int bit_begin, int bit_end, hipStream_t s,
                          bool* result_in_tmp, int nseg) {
    return radix_sort<uint32_t>(keys, vals, tmp_keys, tmp_vals, hist, n, std::min(bit_begin, 32),
                                std::min(bit_end, 32), s, result_in_tmp, nseg);
}

hipError_t exclusive_scan_i32(const int32_t* in, int32_t* out, int64_t n, uint32_t* tile_sums,
                              hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int tiles = (int)sort_tiles(n);
    if (n <= kOwnSumMax) {
        // one launch in place of two: 4 us less for the short rows of small
        // plans.  in and out must not be the same array (nor are they for the
        // larger n, by the callers).
        hipLaunchKernelGGL(scan_tile_apply<kOwnSums>, dim3(tiles), dim3(kThreads), 0, s, in, out, n,
                           tile_sums);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(scan_tile_sums, dim3(tiles), dim3(kThreads), 0, s, in, n, tile_sums);
    if (tiles <= kApplySumMax) {
        hipLaunchKernelGGL(scan_tile_apply<kTileSums>, dim3(tiles), dim3(kThreads), 0, s, in, out, n,
                           tile_sums);
    } else {
        hipLaunchKernelGGL(scan_single, dim3(1), dim3(1024), 0, s, tile_sums, (int64_t)tiles);
        hipLaunchKernelGGL(scan_tile_apply<kScanned>, dim3(tiles), dim3(kThreads), 0, s, in, out, n,
                           tile_sums);
    }
    return hipGetLastError();
}

}  // namespace pmfmm
