// Reverse-mode derivative of the 2D binary64 push: gcb_push_backward.
//
// For a segment of n_steps steps starting from a caller-owned state (taken,
// with its adjoint, into the tile order of the start positions), the host
// recomputes the forward steps with the push kernels (the parity arithmetic of
// the forward pass), keeping the start state of every step and its switch
// decisions.  Then, per batch of steps from the last to the first, the particles
// are cell-sorted by their positions halfway through the batch, the tiles cut
// into chunks, and the particles taken through the batch in reverse
// (gcb_adjoint_kernels.hpp).  The node-interleaved binary64 grid that receives
// the field cotangents is finally added to the caller's dE/dB arrays.
//
// The reverse sweep evaluates its forward values and cotangents in the
// production arithmetic, multiply-adds fused as written (-ffp-contract=on): they
// depend on the forward pass only through the recorded states and decisions.
#define GCB_ARITH_NS arith_fast
#define GCB_FAST_ARITH 1
#include <hip/hip_runtime.h>

#include "gcb_adjoint_kernels.hpp"

namespace gcb {
namespace {

constexpr int kStartsWG = 1024, kStartsPer = 4;

// the contribution of a tile of m particles: chunks in the upper half, loose
// particles in the lower
__device__ __forceinline__ uint64_t tile_share(int m, int part, int few) {
    return m < few ? (uint64_t)m : (uint64_t)((m + part - 1) / part) << 32;
}

// inclusive scan over the workgroup of one value per thread (w: one per wavefront)
__device__ __forceinline__ uint64_t block_scan(uint64_t v, uint64_t* w) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t t = __shfl_up(v, off);
        v += lane >= off ? t : 0;
    }
    if (lane == 63) w[wave] = v;
    __syncthreads();
    for (int i = 0; i < wave; ++i) v += w[i];
    __syncthreads();
    return v;
}

// sums[b] = the share of block b's tiles
__global__ __launch_bounds__(kStartsWG) void k_chunk_sums(const int32_t* __restrict__ tile_start,
                                                          int ntiles, int part, int few,
                                                          uint64_t* sums) {
    __shared__ uint64_t w[kStartsWG / 64];
    const int t0 = ((int)blockIdx.x * kStartsWG + (int)threadIdx.x) * kStartsPer;
    uint64_t v = 0;
#pragma unroll
    for (int i = 0; i < kStartsPer; ++i)
        if (t0 + i < ntiles) v += tile_share(tile_start[t0 + i + 1] - tile_start[t0 + i], part, few);
    v = block_scan(v, w);
    if (threadIdx.x == kStartsWG - 1) sums[blockIdx.x] = v;
}

// the exclusive scan of the shares; sums: those of the blocks (several blocks)
__global__ __launch_bounds__(kStartsWG) void k_chunk_starts(
    const int32_t* __restrict__ tile_start, int ntiles, int part, int few,
    const uint64_t* __restrict__ sums, int32_t* starts, int32_t* loose) {
    __shared__ uint64_t w[kStartsWG / 64];
    __shared__ uint64_t before;
    uint64_t v = 0;
    for (int b = threadIdx.x; b < (int)blockIdx.x; b += kStartsWG) v += sums[b];
    v = block_scan(v, w);
    if (threadIdx.x == kStartsWG - 1) before = v;
    const int t0 = ((int)blockIdx.x * kStartsWG + (int)threadIdx.x) * kStartsPer;
    uint64_t own[kStartsPer], sum = 0;
#pragma unroll
    for (int i = 0; i < kStartsPer; ++i) {
        own[i] = t0 + i < ntiles
                     ? tile_share(tile_start[t0 + i + 1] - tile_start[t0 + i], part, few) : 0;
        sum += own[i];
    }
    uint64_t run = block_scan(sum, w) - sum + before;
#pragma unroll
    for (int i = 0; i < kStartsPer; ++i) {
        if (t0 + i <= ntiles) {
            starts[t0 + i] = (int32_t)(run >> 32);
            loose[t0 + i] = (int32_t)(uint32_t)run;
        }
        run += own[i];
    }
}

// blocks that reach entry ntiles
int starts_blocks(int ntiles) { return ntiles / (kStartsWG * kStartsPer) + 1; }

}  // namespace

int64_t chunk_sums_elems(int ntiles) { return starts_blocks(ntiles); }

hipError_t launch_chunk_starts(const int32_t* tile_start, int ntiles, int part, int few,
                               int32_t* starts, int32_t* loose, uint64_t* sums,
                               hipStream_t stream) {
    const int blocks = starts_blocks(ntiles);
    if (blocks > 1)
        hipLaunchKernelGGL(k_chunk_sums, dim3(blocks), dim3(kStartsWG), 0, stream, tile_start,
                           ntiles, part, few, sums);
    hipLaunchKernelGGL(k_chunk_starts, dim3(blocks), dim3(kStartsWG), 0, stream, tile_start,
                       ntiles, part, few, sums, starts, loose);
    return hipGetLastError();
}

hipError_t launch_adjoint_batch(const AdjointLaunch& L, const PushConst& pc,
                                hipStream_t stream) {
    if (L.n == 0 || L.s_hi <= L.s_lo) return hipSuccess;
    return L.yee ? adj::launch_batch<2, true>(L, pc, stream)
                 : adj::launch_batch<2, false>(L, pc, stream);
}

}  // namespace gcb
