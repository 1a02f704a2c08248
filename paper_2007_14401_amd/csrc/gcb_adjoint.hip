// Reverse-mode derivative of the 2D binary64 push: gcb_push_backward.
//
// For a segment of n_steps steps starting from a caller-owned state (taken,
// with its adjoint, into the tile order of the start positions), the host
// recomputes the forward steps with the push kernels (the parity arithmetic of
// the forward pass), keeping the start state of every step and its switch
// decisions.  Then, per batch of steps from the last to the first, the particles
// are cell-sorted by their positions at the batch's first step, the tiles cut
// into chunks, and one launch takes every particle through the batch in reverse
// (gcb_adjoint_kernels.hpp).  The binary32 node-interleaved grid that receives
// the field cotangents is finally added to the caller's dE/dB arrays.
//
// The reverse sweep evaluates its forward values and cotangents in the
// production arithmetic (compiled with -ffp-contract=fast): they depend on the
// forward pass only through the recorded states and decisions.
#define GCB_ARITH_NS arith_fast
#define GCB_FAST_ARITH 1
#include <hip/hip_runtime.h>

#include "gcb_adjoint_kernels.hpp"

namespace gcb {
namespace {

constexpr int kScanWG = 256;

// starts[t] = chunks of `part` particles of the tiles before t, t in
// [0, ntiles] (one workgroup; a few thousand tiles)
__global__ __launch_bounds__(kScanWG) void k_chunk_starts(
    const int32_t* __restrict__ tile_start, int ntiles, int part, int32_t* starts) {
    __shared__ int s[kScanWG];
    const int per = (ntiles + kScanWG - 1) / kScanWG;
    const int lo = min((int)threadIdx.x * per, ntiles), hi = min(lo + per, ntiles);
    int sum = 0;
    for (int t = lo; t < hi; ++t) sum += (tile_start[t + 1] - tile_start[t] + part - 1) / part;
    s[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < kScanWG; off <<= 1) {
        const int v = (int)threadIdx.x >= off ? s[threadIdx.x - off] : 0;
        __syncthreads();
        s[threadIdx.x] += v;
        __syncthreads();
    }
    int run = s[threadIdx.x] - sum;
    for (int t = lo; t < hi; ++t) {
        starts[t] = run;
        run += (tile_start[t + 1] - tile_start[t] + part - 1) / part;
    }
    if (threadIdx.x == kScanWG - 1) starts[ntiles] = s[threadIdx.x];
}

}  // namespace

hipError_t launch_chunk_starts(const int32_t* tile_start, int ntiles, int part, int32_t* starts,
                               hipStream_t stream) {
    hipLaunchKernelGGL(k_chunk_starts, dim3(1), dim3(kScanWG), 0, stream, tile_start, ntiles,
                       part, starts);
    return hipGetLastError();
}

hipError_t launch_adjoint_batch(const AdjointLaunch& L, const PushConst& pc,
                                hipStream_t stream) {
    if (L.n == 0 || L.s_hi <= L.s_lo) return hipSuccess;
    return L.yee ? adj::launch_batch<2, true>(L, pc, stream)
                 : adj::launch_batch<2, false>(L, pc, stream);
}

}  // namespace gcb
