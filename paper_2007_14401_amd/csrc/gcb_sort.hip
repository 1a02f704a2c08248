// Cell sort of the particle state by tile, so that the particles of a tile
// are contiguous (coalesced structure-of-arrays access) and the tiled push
// kernel can stage one field window per workgroup.
//
// Pipeline (all on the caller's stream), stable.  Up to 256 tiles, or 65536
// with at most kSelfScan blocks of 4096 particles:
//   k_keys_hist    key = tile index; per block the histogram of the key's upper
//                  digit (the bits above the lowest `low`, eight at most)
//   k_scatter      (key, slot) into the buckets of the upper digit: wave-level
//                  multisplit ranks; every block sums the histograms of the
//                  blocks before it itself (more than kSelfScan of them take an
//                  exclusive scan, 3 kernels)
//   k_bucket_sort  a workgroup per bucket: counting sort by the low bits, which
//                  also gives tile_start (with 256 tiles or fewer the scatter
//                  does that, and is the last step); of larger buckets, which
//                  particles gathered in a few tiles make, the counts of their
//                  parts
//   k_bucket_parts those parts, a workgroup each (nothing to do for it costs
//                  1.5 us; not launched where no bucket can be larger)
// Launches and their gaps are most of a sort of 1e5 particles, and the passes
// over the keys of one of 1e6: two to four kernels where an LSD radix sort of
// two digits has twelve (keys; histogram, scan, scatter of each digit; tile
// bounds).  1e6 particles, 2704 tiles: 93 -> 45 us; all of them in one tile 145
// -> 76, half of them 91 -> 66 (1.95 and 0.94 ms with one workgroup per bucket,
// which sorts 16384 particles in some 50 us).
// Otherwise LSD radix sort, 8 bits per pass, and k_tile_bounds: with 256 buckets
// of many particles each the bucket sort has too few wavefronts (1e7 particles,
// 1024 (r, theta) tiles: 12.66 ms of a push with it, 12.44 without).
// The push kernel of the sort's step then reads the state through idx (the
// permutation) and writes it in tile order, so there is no permutation pass
// (the same for the curved-spacetime and 3D states).
// Key2, Key3, KeyGr: the tiles of the 2D, the 3D (cubic) and the
// curved-spacetime state ((r, theta) tiles of the grid cells).
#include <hip/hip_runtime.h>

#include "gcb_internal.h"

namespace gcb {
namespace {

constexpr int kSortWG = 256;
constexpr int kGroups = 4;                 // of 64 particles per wavefront
constexpr int kWaves = 16;                 // per block
constexpr int kItems = kWaves * kGroups * 64;
constexpr int kScanWG = 256;
constexpr int kScanItems = 4096;                          // per block of the scan

// clamped tile coordinate of one position component (non-finite -> 0)
__device__ __forceinline__ int tile_coord(double v, double inv_d, int tile, int nt) {
    const double gc = floor(v * inv_d);
    const int t = (gc >= 0.0 && gc < 2.0e9) ? (int)gc / tile : 0;
    return t < nt ? t : nt - 1;
}

// The key of particle p: its tile, row-major.
struct Key2 {
    const double* x;
    const double* y;
    double inv_dx, inv_dy;
    TileGeom g;
    __device__ uint32_t operator()(int64_t p) const {
        return (uint32_t)(tile_coord(y[p], inv_dy, g.tile, g.nty) * g.ntx +
                          tile_coord(x[p], inv_dx, g.tile, g.ntx));
    }
};

struct Key3 {
    const double* x;
    const double* y;
    const double* z;
    double inv_dx, inv_dy, inv_dz;
    TileGeom3 g;
    __device__ uint32_t operator()(int64_t p) const {
        const int tx = tile_coord(x[p], inv_dx, g.tile, g.ntx);
        const int ty = tile_coord(y[p], inv_dy, g.tile, g.nty);
        const int tz = tile_coord(z[p], inv_dz, g.tile, g.ntz);
        return (uint32_t)((tz * g.nty + ty) * g.ntx + tx);
    }
};

// (r, theta) tile of the particle's grid cell
struct KeyGr {
    const double* r;
    const double* th;
    gr::GrConst g;
    int tile, ntx;
    __device__ uint32_t operator()(int64_t p) const {
        int i, j;
        double wx, wy;
        gr::grid_cell(g, r[p], th[p], i, j, wx, wy);
        return (uint32_t)((j / tile) * ntx + i / tile);
    }
};

// Keys, and per block the histogram of their digits, digit-major (for the scan) or, kByBlock, block by block.
template <bool kByBlock, class Key>
__global__ __launch_bounds__(kWaves * 64) void k_keys_hist(Key key, int64_t n, int shift,
                                                           int nblocks, uint32_t* keys,
                                                           uint32_t* hist) {
    __shared__ uint32_t h[256];
    if (threadIdx.x < 256) h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * (kWaves * kGroups * 64);
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
        const int64_t p = b0 + gi * (kWaves * 64) + threadIdx.x;
        if (p < n) {
            const uint32_t k = key(p);
            keys[p] = k;
            atomicAdd(&h[(k >> shift) & 255u], 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x < 256)
        hist[kByBlock ? (int64_t)blockIdx.x * 256 + threadIdx.x
                      : (int64_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// tile_start[t] = first sorted slot whose key is >= t, for t in [0, ntiles]:
// every slot i writes the starts of the tiles in (key[i-1], key[i]].
__global__ __launch_bounds__(kSortWG) void k_tile_bounds(const uint32_t* __restrict__ keys,
                                                         int64_t n, int ntiles,
                                                         int32_t* tile_start) {
    const int64_t i = (int64_t)blockIdx.x * kSortWG + threadIdx.x;
    if (i > n) return;
    const int lo = i == 0 ? -1 : (int)keys[i - 1];
    const int hi = i == n ? ntiles : (int)keys[i];
    for (int t = lo + 1; t <= hi; ++t) tile_start[t] = (int32_t)i;
}

__global__ __launch_bounds__(kSortWG) void k_radix_hist(const uint32_t* __restrict__ keys,
                                                        int64_t n, int shift,
                                                        int nblocks, uint32_t* hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * kItems;
    for (int e = threadIdx.x; e < kItems; e += kSortWG) {
        const int64_t p = b0 + e;
        if (p < n) atomicAdd(&h[(keys[p] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[(int64_t)threadIdx.x * nblocks + blockIdx.x] = h[threadIdx.x];
}

// exclusive scan, phase 1: block sums
__global__ __launch_bounds__(kScanWG) void k_scan_reduce(const uint32_t* __restrict__ in,
                                                         int64_t n, uint32_t* sums) {
    __shared__ uint32_t s[kScanWG];
    const int64_t b0 = (int64_t)blockIdx.x * kScanItems;
    uint32_t acc = 0;
    for (int e = threadIdx.x; e < kScanItems; e += kScanWG) {
        const int64_t p = b0 + e;
        if (p < n) acc += in[p];
    }
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int off = kScanWG / 2; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) s[threadIdx.x] += s[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) sums[blockIdx.x] = s[0];
}

// block-wide exclusive scan of kScanWG values held one per thread
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* s,
                                                         uint32_t& total) {
    s[threadIdx.x] = v;
    __syncthreads();
    for (int off = 1; off < kScanWG; off <<= 1) {
        const uint32_t t = (int)threadIdx.x >= off ? s[threadIdx.x - off] : 0u;
        __syncthreads();
        s[threadIdx.x] += t;
        __syncthreads();
    }
    total = s[kScanWG - 1];
    const uint32_t incl = s[threadIdx.x];
    __syncthreads();
    return incl - v;
}

// phase 2: exclusive scan of the block sums in one workgroup (any count)
__global__ __launch_bounds__(kScanWG) void k_scan_sums(uint32_t* sums, int nsums) {
    __shared__ uint32_t s[kScanWG];
    uint32_t carry = 0;
    for (int b = 0; b < nsums; b += kScanWG) {
        const int i = b + (int)threadIdx.x;
        const uint32_t v = i < nsums ? sums[i] : 0u;
        uint32_t total;
        const uint32_t ex = block_exclusive_scan(v, s, total);
        if (i < nsums) sums[i] = carry + ex;
        carry += total;
    }
}

// phase 3: scan within each block, offset by its block sum
__global__ __launch_bounds__(kScanWG) void k_scan_down(const uint32_t* __restrict__ in,
                                                       int64_t n,
                                                       const uint32_t* __restrict__ sums,
                                                       uint32_t* out) {
    __shared__ uint32_t s[kScanWG];
    constexpr int kPer = kScanItems / kScanWG;   // contiguous items per thread
    const int64_t b0 = (int64_t)blockIdx.x * kScanItems + (int64_t)threadIdx.x * kPer;
    uint32_t loc[kPer];
    uint32_t acc = 0;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        const int64_t p = b0 + e;
        loc[e] = p < n ? in[p] : 0u;
        acc += loc[e];
    }
    uint32_t total;
    uint32_t run = sums[blockIdx.x] + block_exclusive_scan(acc, s, total);
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        const int64_t p = b0 + e;
        if (p < n) out[p] = run;
        run += loc[e];
    }
}

// exclusive scan of 256 values in LDS by one wavefront
__device__ __forceinline__ void scan_256(uint32_t* v) {
    const int lane = threadIdx.x & 63;
    uint32_t c[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c[i] = v[lane * 4 + i];
        sum += c[i];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(inc, off);
        inc += lane >= off ? t : 0u;
    }
    uint32_t run = inc - sum;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[lane * 4 + i] = run;
        run += c[i];
    }
}

// Rank of each of a wavefront's kGroups x 64 consecutive items (from w0, below
// end) among the items of the same digit, given the counts so far in `count`
// (256 of the wavefront's own, updated).
__device__ __forceinline__ void wave_ranks(const uint32_t* __restrict__ keys, int64_t w0,
                                           int64_t end, int shift, uint32_t mask, int bits,
                                           uint32_t* count, uint32_t rank[kGroups],
                                           uint32_t dig[kGroups]) {
    const int lane = threadIdx.x & 63;
    const unsigned long long lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
        const int64_t p = w0 + gi * 64 + lane;
        dig[gi] = p < end ? (keys[p] >> shift) & mask : 0u;
    }
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
        const bool valid = w0 + gi * 64 + lane < end;
        const uint32_t d = dig[gi];
        unsigned long long peers = __ballot(valid);
        for (int bit = 0; bit < bits; ++bit) {
            const unsigned long long bal = __ballot(valid && ((d >> bit) & 1u));
            peers &= ((d >> bit) & 1u) ? bal : ~bal;
        }
        uint32_t before = 0;
        if (valid) before = count[d];
        // wave-synchronous: every lane has read the counter before the leader updates it
        __builtin_amdgcn_wave_barrier();
        if (valid) {
            const int leader = __ffsll((long long)peers) - 1;
            if (lane == leader) count[d] = before + (uint32_t)__popcll(peers);
        }
        __builtin_amdgcn_wave_barrier();
        rank[gi] = before + (uint32_t)__popcll(peers & lt);
    }
}

// Stable scatter by one digit.  idx null: the slots are 0, 1, 2, ...;
// keys_out null: not kept.  kSelf: hist holds the blocks' histograms
// (k_keys_hist, by block), else their scan.  With `tile_start` the digit is the
// key's upper one, and the buckets' starts are noted at their first tiles.
template <bool kSelf>
__global__ __launch_bounds__(kWaves * 64) void k_scatter(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ idx, int64_t n, int shift,
    int nblocks, const uint32_t* __restrict__ hist, uint32_t* keys_out, uint32_t* idx_out,
    int32_t* tile_start, int ntiles) {
    constexpr int kWG = kWaves * 64;
    __shared__ uint32_t wcount[kWaves][256];
    __shared__ uint32_t gbase[256];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    if constexpr (kSelf) {
        // kWG / 256 threads per digit, each over its share of the blocks; the
        // partial sums meet in wcount
        constexpr int kParts = kWG / 256;
        const int d = threadIdx.x & 255, part = threadIdx.x >> 8;
        uint32_t before = 0, all = 0;
#pragma unroll 16
        for (int b = part; b < nblocks; b += kParts) {
            const uint32_t v = hist[b * 256 + d];
            before += b < (int)blockIdx.x ? v : 0u;
            all += v;
        }
        wcount[part][d] = before;
        wcount[kParts + part][d] = all;
        __syncthreads();
        if (threadIdx.x < 256) {
            before = all = 0;
#pragma unroll
            for (int i = 0; i < kParts; ++i) {
                before += wcount[i][d];
                all += wcount[kParts + i][d];
            }
            gbase[d] = all;
        }
        __syncthreads();
        if (wave == 0) scan_256(gbase);
        __syncthreads();
        if (threadIdx.x < 256) gbase[d] += before;
        __syncthreads();
    } else if (threadIdx.x < 256) {
        gbase[threadIdx.x] = hist[(int64_t)threadIdx.x * nblocks + blockIdx.x];
    }
    if (tile_start && blockIdx.x == 0 && threadIdx.x < 256) {
        const int64_t t = (int64_t)threadIdx.x << shift;
        if (t < ntiles) tile_start[t] = (int32_t)gbase[threadIdx.x];
        if (threadIdx.x == 0) tile_start[ntiles] = (int32_t)n;
    }
    for (int d = threadIdx.x; d < 256 * kWaves; d += kWG) (&wcount[0][0])[d] = 0;
    __syncthreads();

    const int64_t w0 = ((int64_t)blockIdx.x * kWaves + wave) * (kGroups * 64);
    uint32_t rank[kGroups];
    uint32_t dig[kGroups];
    wave_ranks(keys, w0, n, shift, 255u, 8, wcount[wave], rank, dig);
    __syncthreads();
    // exclusive prefix of the per-wave counts, per digit
    if (threadIdx.x < 256) {
        const int d = threadIdx.x;
        uint32_t run = gbase[d];
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = wcount[w][d];
            wcount[w][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int gi = 0; gi < kGroups; ++gi) {
        const int64_t p = w0 + gi * 64 + lane;
        if (p < n) {
            const uint32_t dst = wcount[wave][dig[gi]] + rank[gi];
            if (keys_out) keys_out[dst] = keys[p];
            idx_out[dst] = idx ? idx[p] : (uint32_t)p;
        }
    }
}

constexpr int kBucketWG = 1024;
constexpr int kBucketMost = 16384;   // particles of a bucket that one workgroup sorts
constexpr int kPart = 8192;          // those of a larger one that a workgroup takes

// The particles [s, e) of a bucket to their places by the low bits of their keys:
// base[d] the next place of digit d (LDS, of 256).
__device__ __forceinline__ void place_by_low(const uint32_t* __restrict__ keys,
                                             const uint32_t* __restrict__ idx, int64_t s,
                                             int64_t e, int low, uint32_t* base,
                                             uint32_t (*wcount)[256], uint32_t* idx_out) {
    constexpr int kWaves = kBucketWG / 64, kChunk = kBucketWG * kGroups;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    for (int64_t c0 = s; c0 < e; c0 += kChunk) {
        __syncthreads();
        for (int d = threadIdx.x; d < 256 * kWaves; d += kBucketWG) (&wcount[0][0])[d] = 0;
        __syncthreads();
        const int64_t w0 = c0 + wave * (kGroups * 64);
        uint32_t rank[kGroups];
        uint32_t dig[kGroups];
        wave_ranks(keys, w0, e, 0, (1u << low) - 1u, low, wcount[wave], rank, dig);
        __syncthreads();
        if (threadIdx.x < 256) {
            const int d = threadIdx.x;
            uint32_t run = base[d];
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const uint32_t c = wcount[w][d];
                wcount[w][d] = run;
                run += c;
            }
            base[d] = run;
        }
        __syncthreads();
#pragma unroll
        for (int gi = 0; gi < kGroups; ++gi) {
            const int64_t p = w0 + gi * 64 + lane;
            if (p < e) idx_out[wcount[wave][dig[gi]] + rank[gi]] = idx[p];
        }
    }
}

// counts of the low bits of the keys of [s, e), in LDS (256)
__device__ __forceinline__ void count_low(const uint32_t* __restrict__ keys, int64_t s, int64_t e,
                                          int low, uint32_t* count) {
    if (threadIdx.x < 256) count[threadIdx.x] = 0;
    __syncthreads();
    for (int64_t p = s + threadIdx.x; p < e; p += kBucketWG)
        atomicAdd(&count[keys[p] & ((1u << low) - 1u)], 1u);
    __syncthreads();
}

// the starts of a bucket's tiles but the first, from t0 + 1 on
__device__ __forceinline__ void note_starts(const uint32_t* base, int low, int t0, int ntiles,
                                            int32_t* tile_start) {
    const int d = threadIdx.x;
    if (d > 0 && d < (1 << low) && t0 + d < ntiles) tile_start[t0 + d] = (int32_t)base[d];
}

// A part of a bucket of more than kBucketMost particles: the i-th over all such
// buckets.  `first` is the number of the bucket's first part, `parts` how many
// it has (0: there are not so many parts).  Called by the whole workgroup.
struct BucketPart {
    int t0, first, parts;
    int64_t s, e;   // the part's particles
    int64_t s0;     // the bucket's first

    __device__ void find(int i, const int32_t* tile_start, int64_t n, int low, int ntiles,
                         uint32_t* before /* LDS, 257 */, uint32_t* total) {
        const int buckets = ((ntiles - 1) >> low) + 1;
        const int b = threadIdx.x;
        auto start = [&](int k) -> int64_t { return k < buckets ? tile_start[k << low] : n; };
        if (b < 256) {
            const int64_t m = b < buckets ? start(b + 1) - start(b) : 0;
            before[b] = m > kBucketMost ? (uint32_t)((m + kPart - 1) / kPart) : 0u;
            if (b == 255) before[256] = before[255];
        }
        __syncthreads();
        if (b < 64) scan_256(before);
        __syncthreads();
        if (b == 0) before[256] += before[255];
        __syncthreads();
        *total = before[256];
        parts = 0;
        if (i >= (int)before[256]) return;
        int lo = 0, hi = 256;   // before[lo] <= i < before[hi]
        while (hi - lo > 1) {
            const int h = (lo + hi) >> 1;
            if ((int)before[h] <= i) lo = h; else hi = h;
        }
        first = (int)before[lo];
        parts = (int)before[lo + 1] - first;
        t0 = lo << low;
        s0 = start(lo);
        s = s0 + (int64_t)(i - first) * kPart;
        e = min(s + kPart, start(lo + 1));
    }
};

// Counting sort of one bucket (the particles of the 2^low tiles from
// blockIdx.x << low) by the low bits, and the starts of its tiles.  Larger buckets
// (particles gathered in few tiles) are left to k_bucket_parts; the workgroups
// after the buckets' count their parts' low bits for it (part_hist) and how many
// parts there are (*nparts).
__global__ __launch_bounds__(kBucketWG) void k_bucket_sort(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ idx, int64_t n, int low,
    int ntiles, int32_t* tile_start, uint32_t* idx_out, uint32_t* part_hist, uint32_t* nparts) {
    __shared__ uint32_t wcount[kBucketWG / 64][256];
    __shared__ uint32_t base[257];
    const int buckets = ((ntiles - 1) >> low) + 1;
    if ((int)blockIdx.x >= buckets) {
        BucketPart part;
        uint32_t total;
        const int i = (int)blockIdx.x - buckets;
        part.find(i, tile_start, n, low, ntiles, base, &total);
        if (i == 0 && threadIdx.x == 0) *nparts = total;
        if (part.parts == 0) return;
        __syncthreads();
        count_low(keys, part.s, part.e, low, base);
        if (threadIdx.x < 256) part_hist[(int64_t)i * 256 + threadIdx.x] = base[threadIdx.x];
        return;
    }
    const int t0 = (int)blockIdx.x << low;
    const int64_t s = tile_start[t0];
    const int64_t e = t0 + (1 << low) < ntiles ? tile_start[t0 + (1 << low)] : n;
    if (e - s > kBucketMost) return;
    count_low(keys, s, e, low, base);
    if (threadIdx.x < 64) scan_256(base);
    __syncthreads();
    if (threadIdx.x < 256) {
        base[threadIdx.x] += (uint32_t)s;
        note_starts(base, low, t0, ntiles, tile_start);
    }
    place_by_low(keys, idx, s, e, low, base, wcount, idx_out);
}

// The parts of the buckets that k_bucket_sort leaves, a workgroup each: the counts
// of the bucket's parts give it its places.
__global__ __launch_bounds__(kBucketWG) void k_bucket_parts(
    const uint32_t* __restrict__ keys, const uint32_t* __restrict__ idx, int64_t n, int low,
    int ntiles, int32_t* tile_start, uint32_t* idx_out, const uint32_t* __restrict__ part_hist,
    const uint32_t* __restrict__ nparts) {
    if (blockIdx.x >= *nparts) return;
    __shared__ uint32_t wcount[kBucketWG / 64][256];
    __shared__ uint32_t base[257];
    BucketPart part;
    uint32_t total;
    const int i = (int)blockIdx.x;
    part.find(i, tile_start, n, low, ntiles, base, &total);
    __syncthreads();
    const int d = threadIdx.x;
    uint32_t before = 0, all = 0;
    if (d < 256) {
        for (int k = 0; k < part.parts; ++k) {
            const uint32_t c = part_hist[(int64_t)(part.first + k) * 256 + d];
            before += part.first + k < i ? c : 0u;
            all += c;
        }
        base[d] = all;
    }
    __syncthreads();
    if (d < 64) scan_256(base);
    __syncthreads();
    if (d < 256) {
        base[d] += (uint32_t)part.s0;
        if (i == part.first) note_starts(base, low, part.t0, ntiles, tile_start);
        base[d] += before;
    }
    place_by_low(keys, idx, part.s, part.e, low, base, wcount, idx_out);
}

hipError_t scan_exclusive(const uint32_t* in, uint32_t* out, int64_t n, uint32_t* sums,
                          hipStream_t stream) {
    const int nb = (int)((n + kScanItems - 1) / kScanItems);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kScanWG), 0, stream, in, n, sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(kScanWG), 0, stream, sums, nb);
    hipLaunchKernelGGL(k_scan_down, dim3(nb), dim3(kScanWG), 0, stream, in, n, sums, out);
    return hipGetLastError();
}

}  // namespace

namespace {

constexpr int kMaxBucketBits = 16;   // an upper digit of 8 bits, a lower of 8
constexpr int kSelfScan = 256;       // blocks whose histograms a scatter sums

int key_bits(int ntiles) {
    int nbits = 0;
    while (((int64_t)1 << nbits) < ntiles) ++nbits;
    return nbits;
}

// keys and the scatter by the digit at `shift`; `upper`: the upper digit
template <bool kSelf, class Key>
hipError_t first_pass(const Key& key, int64_t n, int shift, uint32_t* kin, uint32_t* kout,
                      uint32_t* iout, int ntiles, bool upper, const SortBuffers& b,
                      hipStream_t stream) {
    const int nblocks = (int)((n + kItems - 1) / kItems);
    hipLaunchKernelGGL((k_keys_hist<kSelf, Key>), dim3(nblocks), dim3(kWaves * 64), 0,
                       stream, key, n, shift, nblocks, kin, b.hist);
    if constexpr (!kSelf) {
        hipError_t e = scan_exclusive(b.hist, b.hist, 256ll * nblocks, b.scan_tmp, stream);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_scatter<kSelf>, dim3(nblocks), dim3(kWaves * 64), 0, stream,
                       kin, nullptr, n, shift, nblocks, b.hist, kout, iout,
                       upper ? b.tile_start : nullptr, ntiles);
    return hipGetLastError();
}

hipError_t tile_bounds(const uint32_t* keys, int64_t n, int ntiles, const SortBuffers& b,
                       hipStream_t stream) {
    const unsigned blocks = (unsigned)((n + 1 + kSortWG - 1) / kSortWG);
    hipLaunchKernelGGL(k_tile_bounds, dim3(blocks), dim3(kSortWG), 0, stream, keys, n, ntiles,
                       b.tile_start);
    return hipGetLastError();
}

// b.idx = the stable order of the particles by key, b.tile_start their starts
template <class Key>
hipError_t cell_sort(const Key& key, int64_t n, int ntiles, const SortBuffers& b,
                     hipStream_t stream) {
    if (n == 0) return tile_bounds(b.keys, n, ntiles, b, stream);
    const int nbits = key_bits(ntiles);
    const int nblocks = (int)((n + kItems - 1) / kItems);
    hipError_t e;
    if (nbits <= 8 || (nbits <= kMaxBucketBits && nblocks <= kSelfScan)) {
        const int low = nbits > 8 ? nbits - 8 : 0;
        uint32_t* kout = low ? b.keys2 : nullptr;
        uint32_t* iout = low ? b.idx2 : b.idx;
        e = nblocks <= kSelfScan
                ? first_pass<true>(key, n, low, b.keys, kout, iout, ntiles, true, b, stream)
                : first_pass<false>(key, n, low, b.keys, kout, iout, ntiles, true, b, stream);
        if (e != hipSuccess || !low) return e;
        const int buckets = ((ntiles - 1) >> low) + 1;
        // parts of large buckets: full ones and a rest of each
        const int parts = n > kBucketMost ? (int)(n / kPart + n / kBucketMost) : 0;
        hipLaunchKernelGGL(k_bucket_sort, dim3(buckets + parts), dim3(kBucketWG), 0, stream,
                           kout, iout, n, low, ntiles, b.tile_start, b.idx, b.hist, b.scan_tmp);
        if (parts)
            hipLaunchKernelGGL(k_bucket_parts, dim3(parts), dim3(kBucketWG), 0, stream, kout,
                               iout, n, low, ntiles, b.tile_start, b.idx, b.hist, b.scan_tmp);
        return hipGetLastError();
    }
    // LSD, the last pass into b.idx
    const int passes = (nbits + 7) / 8;
    uint32_t* ks[2] = {b.keys, b.keys2};
    uint32_t* is[2] = {b.idx, b.idx2};
    e = first_pass<false>(key, n, 0, ks[passes & 1], ks[(passes - 1) & 1],
                          is[(passes - 1) & 1], ntiles, false, b, stream);
    if (e != hipSuccess) return e;
    for (int p = 1; p < passes; ++p) {
        const int in = (passes - p) & 1, out = in ^ 1;
        hipLaunchKernelGGL(k_radix_hist, dim3(nblocks), dim3(kSortWG), 0, stream, ks[in], n,
                           8 * p, nblocks, b.hist);
        e = scan_exclusive(b.hist, b.hist, 256ll * nblocks, b.scan_tmp, stream);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_scatter<false>, dim3(nblocks), dim3(kWaves * 64), 0, stream,
                           ks[in], is[in], n, 8 * p, nblocks, b.hist, ks[out], is[out], nullptr,
                           ntiles);
    }
    return tile_bounds(ks[0], n, ntiles, b, stream);
}

}  // namespace

int64_t sort_hist_elems(int64_t n) {
    const int64_t nblocks = (n + kItems - 1) / kItems;
    return 256 * (nblocks > 0 ? nblocks : 1);
}

int64_t sort_scan_tmp_elems(int64_t n_scan) { return (n_scan + kScanItems - 1) / kScanItems + 1; }

hipError_t launch_cell_sort(const double* x, const double* y, int64_t n, double inv_dx,
                            double inv_dy, const TileGeom& g, const SortBuffers& b,
                            hipStream_t stream) {
    return cell_sort(Key2{x, y, inv_dx, inv_dy, g}, n, g.ntx * g.nty, b, stream);
}

hipError_t launch_gr_cell_sort(const double* r, const double* th, int64_t n,
                               const gr::GrConst& g, int tile, const SortBuffers& b,
                               hipStream_t stream) {
    const int ntx = (g.nr + tile - 1) / tile, nty = (g.nth + tile - 1) / tile;
    return cell_sort(KeyGr{r, th, g, tile, ntx}, n, ntx * nty, b, stream);
}

hipError_t launch_cell_sort3(const double* x, const double* y, const double* z, int64_t n,
                             double inv_dx, double inv_dy, double inv_dz, const TileGeom3& g,
                             const SortBuffers& b, hipStream_t stream) {
    return cell_sort(Key3{x, y, z, inv_dx, inv_dy, inv_dz, g}, n, g.ntx * g.nty * g.ntz, b,
                     stream);
}

}  // namespace gcb
