// Kernel of the reverse sweep, for D = 2 or 3 dimensions.
//
// A batch of steps is one launch.  Particles are independent, so a lane takes
// a particle through all steps of the batch in reverse order with its cotangents
// in registers; nothing but the start states and the decisions is read per step
// and nothing written.  A workgroup takes the particles of one tile of a cell
// sort (or a part of a crowded tile's) and keeps W^D nodes around the tile in
// LDS: the fields, and the sums of the node cotangents, which are added to the
// gradient grid once at the end.  The window reaches as far as a particle can
// drift in the batch; what falls outside all the same goes to the grid directly.
// Particles of nearly empty tiles have a kernel without windows (k_adjoint_loose).
//
// Node sums in binary64, because the LDS adds those at full speed and binary32
// ones lane by lane: a wavefront's ds_add_f32 holds the LDS for 194 cycles
// wherever its addresses lie, ds_add_f64 for 12 (consecutive) to 22 (random).
// With binary32 sums the 2D sweep below took 20.5 ms instead of 6.3 (its tiles of
// 30 then).
// Device-scope atomics, some 2e10 per second with an address per lane, are slower
// again: hence the window.
//
// Bound by the LDS in 2D (72 % busy: at K = 4 a guiding-center step has six points
// of 24 adds and eleven gathers of 16 loads; VALU 56 %) with two wavefronts per
// SIMD to hide its latency: 256 registers and the window leave room for no
// more.  In 3D a window's tile has 216 cells, whose particles need not fill the
// wavefronts (225 of them at 3e5 on 64^3: LDS 43 %, VALU 30 %).
//   2D, 1e6 particles, 1024^2, 32 steps, K = 4: 5.9 ms, the whole backward 35.1
//   -> 10.3 ms, 9.7 with the sorts of today (before: a launch per step and
//   regime with global gathers, records of the cotangents to memory, and their
//   scatter: 18.5 and 11.7 ms).
//   3D, 3e5 particles, 64^3, 8 steps: 1.6 ms; training step 8.6 -> 4.7 ms, 4.0
//   with the sorts and staging of today.
// Tiles of 32 in a window of 40 (2D; 28: 11.4 ms, 30: 10.7, 32: 10.3; two
// workgroups of four wavefronts with windows of 28: 10.5) and of 6 in 11 (3D;
// 5: 5.7 ms, 6: 4.7, 7: 5.1).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>

#include "gcb_adjoint.hpp"
#include "gcb_internal.h"
#include "gcb_queues.hpp"

namespace gcb {
namespace adj {

// *p += v for a value of the gradient grid, by the memory's own addition
__device__ __forceinline__ void grid_add(double* p, double v) {
    __builtin_amdgcn_global_atomic_fadd_f64(
        (__attribute__((address_space(1))) double*)p, v);
}

// Node cotangents: W^D nodes of six components in LDS, a plane per component,
// covering global nodes [o, o + W) per axis (periodic).
template <int D>
struct Window {
    static constexpr int W = kAdjWindow<D>;
    static constexpr int kPlane = D == 2 ? W * W : W * W * W;
    double* lds;
    double* grad;   // node-interleaved grid
    int o[D], n[D];

    __device__ void node(int k, const int c[D], double v) const {
        int e = 0;
        bool in = true;
#pragma unroll
        for (int a = D - 1; a >= 0; --a) {
            int d = c[a] - o[a];
            if ((unsigned)d >= (unsigned)W) d += d < 0 ? n[a] : -n[a];
            in = in && (unsigned)d < (unsigned)W;
            e = e * W + d;
        }
        if (in) {
            atomicAdd(lds + k * kPlane + e, v);
        } else {
            size_t g = 0;
#pragma unroll
            for (int a = D - 1; a >= 0; --a) g = g * n[a] + wrap_index(c[a], n[a]);
            grid_add(grad + g * 6 + k, v);
        }
    }

    template <bool kYee>
    __device__ void add(const typename Dim<D>::Push& pc, const double X[D],
                        const Point<D, kYee>& p, const SampleBar<D>& sb) const {
        constexpr int kC = 1 << D;
        if (__builtin_expect(p.in, 1)) {
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                double q[kC];
                nodes_back(p, sb, k, q);
                double* w = lds + k * kPlane + p.off[k];
#pragma unroll
                for (int c = 0; c < kC; ++c)
                    atomicAdd(w + (c & 1) + ((c >> 1) & 1) * W + (D == 3 ? (c >> 2) * W * W : 0),
                              q[c]);
            }
        } else {
            // a stencil at the window's edge or beyond: node by node
            Point<D, kYee> t;
            int cell[D][Point<D, kYee>::kSets];
            place<D>(pc, X, cell, t);
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                double q[kC];
                nodes_back(p, sb, k, q);
#pragma unroll 1
                for (int c = 0; c < kC; ++c) {
                    int i[D];
#pragma unroll
                    for (int a = 0; a < D; ++a) i[a] = cell[a][p.entry(k, a)] + ((c >> a) & 1);
                    double v = q[0];
#pragma unroll
                    for (int b = 1; b < kC; ++b) v = c == b ? q[b] : v;
                    if (v != 0.0) node(k, i, v);
                }
            }
        }
    }
};

// element of the node-interleaved grid at which row `row` of a window's nodes
// starts (at global column 0)
template <int D>
__device__ __forceinline__ size_t grid_row(const Window<D>& w, int row) {
    size_t g = wrap_index(w.o[1] + row % Window<D>::W, w.n[1]);
    if (D == 3) g += (size_t)wrap_index(w.o[D - 1] + row / Window<D>::W, w.n[D - 1]) * w.n[1];
    return g * w.n[0] * 6;
}

// particle p through the steps [s_lo, s_hi) of a segment, last to first
template <int D, bool kYee, class Acc, class Win>
__device__ __forceinline__ void sweep_particle(
    const Acc& acc, const Win& win, const typename Dim<D>::Push& pc,
    const typename Dim<D>::Const& K, int64_t p, const double* __restrict__ rec,
    const double* __restrict__ qm_arr, const uint8_t* __restrict__ S, double* lam, int64_t n,
    int s_lo, int s_hi) {
    constexpr int kL = 2 * D + 3;
    const double qm = qm_arr ? qm_arr[p] : Dim<D>::base(pc).qm;
    double l[kL];
#pragma unroll
    for (int c = 0; c < kL; ++c) l[c] = lam[c * n + p];
    for (int s = s_hi - 1; s >= s_lo; --s) {
        const double* r = rec + (size_t)s * kL * n + p;
        double st[kL];
#pragma unroll
        for (int c = 0; c < kL; ++c) st[c] = r[c * n];
        if (S[(size_t)s * n + p] == 0)
            gca_vjp<D, kYee>(acc, win, pc, K, st, qm, l);
        else
            boris_vjp<D, kYee>(acc, win, pc, K, st, qm, l);
    }
#pragma unroll
    for (int c = 0; c < kL; ++c) lam[c * n + p] = l[c];
}

// Node cotangents of a wavefront's lanes, each to its own place in the grid: the
// lanes of a call put their values into LDS (kPoints of them at a time) and then
// add them together, so that neighbouring lanes add to neighbouring components
// and nodes of one point, and an atomic instruction reaches a few cache lines
// instead of one per lane.  All six components of a point at a time: three by
// three they reach twice the lines (256^3, 1e6 particles, 4 steps: 21.2 -> 15.8 ms).
template <int D, bool kYee>
struct LaneSums {
    static constexpr int kC = 1 << D;
    static constexpr int kV = 6 * kC;                 // values of a point
    static constexpr int kStride = kV + 1;            // in LDS
    static constexpr int kPoints = D == 2 ? 64 : 32;
    static constexpr int kSets = Point<D, kYee>::kSets;
    static constexpr size_t kBytes =
        kPoints * (kStride * sizeof(double) + D * kSets * sizeof(int));
    double* val;   // kPoints x kStride, of the wavefront's own
    int* cell;     // kPoints x D x kSets
    double* grad;
    int n[D];

    template <bool kY>
    __device__ void add(const typename Dim<D>::Push& pc, const double X[D],
                        const Point<D, kY>& p, const SampleBar<D>& sb) const {
        static_assert(kY == kYee, "the lattice of the kernel");
        // the lanes of this call, numbered
        const unsigned long long here = __ballot(1);
        const int lanes = __popcll(here);
        const int rank = __popcll(here & ((1ull << (threadIdx.x & 63)) - 1ull));
        for (int first = 0; first < lanes; first += kPoints) {
            const int own = rank - first;
            if ((unsigned)own < (unsigned)kPoints) {
                Point<D, kYee> t;
                int c[D][kSets];
                place<D>(pc, X, c, t);
#pragma unroll
                for (int a = 0; a < D; ++a)
#pragma unroll
                    for (int s = 0; s < kSets; ++s)
                        cell[(own * D + a) * kSets + s] = wrap_index(c[a][s], n[a]);
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    double q[kC];
                    nodes_back(p, sb, k, q);
#pragma unroll
                    for (int i = 0; i < kC; ++i) val[own * kStride + i * 6 + k] = q[i];
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int all = min(kPoints, lanes - first) * kV;
#pragma unroll 4
            for (int e = rank; e < all; e += lanes) {
                const int pt = e / kV, u = e - pt * kV;
                const int corner = u / 6, k = u - corner * 6;
                const double v = val[pt * kStride + u];
                size_t g = 0;
#pragma unroll
                for (int a = D - 1; a >= 0; --a) {
                    const int s = kYee ? (Dim<D>::packed_sets() >> (3 * k + a)) & 1 : k;
                    int m = cell[(pt * D + a) * kSets + s] + ((corner >> a) & 1);
                    m = m == n[a] ? 0 : m;
                    g = g * n[a] + m;
                }
                if (v != 0.0) grid_add(grad + g * 6 + k, v);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        }
    }
};

// The wavefronts of a workgroup take the slices of 64 of its two queues (see
// split_queues): nG of m entries in the first.  Each its own to begin with, so
// that the long ones in front go to different SIMDs (300 particles per tile: 757
// us of a sweep with the first come first served, 625 so), then the next
// (*next_slice: 0).
template <class Sweep>
__device__ __forceinline__ void take_slices(int nG, int m, int* next_slice, Sweep&& sweep) {
    const int lane = threadIdx.x & 63;
    const int waves = blockDim.x >> 6;
    const int sG = (nG + 63) >> 6;
    const int sAll = sG + ((m - nG + 63) >> 6);
    int sl = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    while (sl < sAll) {
        const bool gslice = sl < sG;
        const int q = gslice ? sl * 64 + lane : nG + (sl - sG) * 64 + lane;
        if (q < (gslice ? nG : m)) sweep(q);
        if (lane == 0) sl = waves + atomicAdd(next_slice, 1);
        sl = __builtin_amdgcn_readfirstlane(sl);
    }
}

// One workgroup per chunk of a tile's particles (chunk c of the launch: tile
// t with starts[t] <= c < starts[t+1], particles [c - starts[t]] * part of the
// tile's), for the steps [s_lo, s_hi) of a segment, last to first.  Slot p of
// the sort is particle perm[p]; rec holds the start states of all the segment's
// steps, S their decisions.
template <int D, bool kYee>
__global__ __launch_bounds__(kAdjWG) __attribute__((amdgpu_waves_per_eu(2))) void
k_adjoint_batch(const double* __restrict__ rec, const double* __restrict__ qm_arr,
                const uint8_t* __restrict__ S, const uint32_t* __restrict__ perm,
                const int32_t* __restrict__ tile_start, const int32_t* __restrict__ starts,
                int ntx, int nty, int ntiles, int tile, int part, double* lam, int64_t n,
                int s_lo, int s_hi, const double* __restrict__ F, typename Dim<D>::Push pc,
                double* grad) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int wave_g[kAdjWG / 64];
    __shared__ int wave_b[kAdjWG / 64];
    __shared__ int next_slice;
    constexpr int W = Window<D>::W;
    constexpr int kAll = 6 * Window<D>::kPlane;

    // consecutive chunks on the same XCD (workgroup b runs on XCD b % 8)
    const int total = starts[ntiles];
    const int per = (total + 7) / 8;
    const int turn = (int)(blockIdx.x / 8);
    if (turn >= per) return;
    const int chunk = (int)(blockIdx.x % 8) * per + turn;
    if (chunk >= total) return;
    double* F_lds = reinterpret_cast<double*>(smem);
    double* win_lds = F_lds + kAll;
    uint16_t* queue = reinterpret_cast<uint16_t*>(win_lds + kAll);

    int t0 = 0, t1 = ntiles;   // starts[t0] <= chunk < starts[t1]
    while (t1 - t0 > 1) {
        const int m = (t0 + t1) >> 1;
        if (starts[m] <= chunk) t0 = m; else t1 = m;
    }
    const int p0 = tile_start[t0] + (chunk - starts[t0]) * part;
    const int p1 = min(tile_start[t0 + 1], p0 + part);
    const int m = p1 - p0;

    Window<D> win;
    win.lds = win_lds;
    win.grad = grad;
    const int tc[3] = {t0 % ntx, D == 2 ? t0 / ntx : (t0 / ntx) % nty, t0 / (ntx * nty)};
#pragma unroll
    for (int a = 0; a < D; ++a) {
        win.o[a] = tc[a] * tile - (W - tile) / 2;
        win.n[a] = Dim<D>::nodes(pc, a);
    }
    const typename Dim<D>::Acc acc = Dim<D>::acc(F_lds, F, pc, win.o, W);

    // stage the fields: rows of W records (6 W values, contiguous in the
    // node-interleaved array) by wavefronts, the loads of kFlight of them in
    // flight together
    constexpr int kRows = kAll / (6 * W), kCols = (6 * W + 63) / 64, kFlight = D == 2 ? 5 : 8;
    int goff[kCols], loff[kCols], lrow[kCols];
#pragma unroll
    for (int u = 0; u < kCols; ++u) {
        const int e = (threadIdx.x & 63) + 64 * u;
        const int c = e / 6, k = e - 6 * c;
        goff[u] = e < 6 * W ? wrap_index(win.o[0] + c, win.n[0]) * 6 + k : -1;
        loff[u] = D == 2 ? window_elem<double>(k, c, W * W) : k * Window<D>::kPlane + c;
        lrow[u] = W * (D == 2 ? window_step<double>(k) : 1);
    }
    for (int row0 = threadIdx.x >> 6; row0 < kRows; row0 += kFlight * (kAdjWG / 64)) {
        double v[kFlight][kCols];
#pragma unroll
        for (int r = 0; r < kFlight; ++r) {
            const int row = row0 + r * (kAdjWG / 64);
            if (row < kRows) {
                const double* src = F + grid_row(win, row);
#pragma unroll
                for (int u = 0; u < kCols; ++u) v[r][u] = goff[u] >= 0 ? src[goff[u]] : 0.0;
            }
        }
#pragma unroll
        for (int r = 0; r < kFlight; ++r) {
            const int row = row0 + r * (kAdjWG / 64);
#pragma unroll
            for (int u = 0; u < kCols; ++u)
                if (row < kRows && goff[u] >= 0) F_lds[loff[u] + row * lrow[u]] = v[r][u];
        }
    }
    for (int e = threadIdx.x; e < kAll; e += kAdjWG) win_lds[e] = 0.0;
    if (threadIdx.x == 0) next_slice = 0;
    // particles of the same regime to the same wavefronts, as in the push
    const uint8_t* Slast = S + (size_t)(s_hi - 1) * n;
    const int nG = split_queues<kAdjWG>(m, queue, wave_g, wave_b,
                                        [&](int q) { return Slast[perm[p0 + q]] == 0; });
    __syncthreads();
    const typename Dim<D>::Const K = Dim<D>::consts(pc);
    take_slices(nG, m, &next_slice, [&](int q) {
        sweep_particle<D, kYee>(acc, win, pc, K, perm[p0 + queue[q]], rec, qm_arr, S, lam, n, s_lo,
                                s_hi);
    });
    __syncthreads();
    // the window to the grid, the values of a row of nodes by neighbouring lanes
    for (int row = threadIdx.x >> 6; row < kRows; row += kAdjWG / 64) {
        double* dst = grad + grid_row(win, row);
        for (int e = threadIdx.x & 63; e < 6 * W; e += 64) {
            const int c = e / 6, k = e - 6 * c;
            const double v = win_lds[(k * kRows + row) * W + c];
            if (v != 0.0) grid_add(dst + wrap_index(win.o[0] + c, win.n[0]) * 6 + k, v);
        }
    }
}

// The same for the particles of tiles with few of them (loose[t]: such particles
// in the tiles before t), `part` per workgroup in the order of the sort: a
// window of LDS and a workgroup would serve a few lanes there, so these gather
// from the grid and add to it.  Bound by those additions once the device is full
// (5e10 per second), by the latency of a step below.  A particle's bits are those
// of the other kernel: the same source, with multiply-adds fused as it is written
// (-ffp-contract=on).
//   3D, 256^3, 1e5 particles, 4 steps: 19.9 ms with a window per tile, 2.0 here;
//   2D, 4096^2, 1e5, 8 steps: 7.8 and 1.4 ms.
template <int D, bool kYee>
__global__ __launch_bounds__(kLooseWG) __attribute__((amdgpu_waves_per_eu(2))) void
k_adjoint_loose(const double* __restrict__ rec, const double* __restrict__ qm_arr,
                const uint8_t* __restrict__ S, const uint32_t* __restrict__ perm,
                const int32_t* __restrict__ tile_start, const int32_t* __restrict__ loose,
                int ntiles, int part, double* lam, int64_t n, int s_lo, int s_hi,
                const double* __restrict__ F, typename Dim<D>::Push pc, double* grad) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int wave_g[kLooseWG / 64];
    __shared__ int wave_b[kLooseWG / 64];
    __shared__ int next_slice;
    __shared__ uint32_t id[kLoosePart];
    __shared__ uint16_t queue[kLoosePart];
    // consecutive chunks on the same XCD, as above
    const int total = loose[ntiles];
    const int per = ((total + part - 1) / part + 7) / 8;
    const int turn = (int)(blockIdx.x / 8);
    if (turn >= per) return;
    const int64_t at0 = ((int64_t)(blockIdx.x % 8) * per + turn) * part;
    if (at0 >= total) return;
    const int first = (int)at0;
    const int m = min(part, total - first);

    LaneSums<D, kYee> sums;
    unsigned char* own = smem + (threadIdx.x >> 6) * LaneSums<D, kYee>::kBytes;
    sums.val = reinterpret_cast<double*>(own);
    sums.cell = reinterpret_cast<int*>(sums.val + LaneSums<D, kYee>::kPoints * LaneSums<D, kYee>::kStride);
    sums.grad = grad;
#pragma unroll
    for (int a = 0; a < D; ++a) sums.n[a] = Dim<D>::nodes(pc, a);
    const typename Dim<D>::Direct acc = Dim<D>::direct(F, pc);

    if (threadIdx.x == 0) next_slice = 0;
    const uint8_t* Slast = S + (size_t)(s_hi - 1) * n;
    const int nG = split_queues<kLooseWG>(m, queue, wave_g, wave_b, [&](int q) {
        const int at = first + q;
        int t0 = 0, t1 = ntiles;   // loose[t0] <= at < loose[t1]
        while (t1 - t0 > 1) {
            const int h = (t0 + t1) >> 1;
            if (loose[h] <= at) t0 = h; else t1 = h;
        }
        const uint32_t p = perm[tile_start[t0] + (at - loose[t0])];
        id[q] = p;
        return Slast[p] == 0;
    });
    __syncthreads();
    const typename Dim<D>::Const K = Dim<D>::consts(pc);
    take_slices(nG, m, &next_slice, [&](int q) {
        sweep_particle<D, kYee>(acc, sums, pc, K, id[queue[q]], rec, qm_arr, S, lam, n, s_lo,
                                s_hi);
    });
}

template <int D, bool kYee>
hipError_t launch_batch(const AdjointLaunch& L, const typename Dim<D>::Push& pc,
                        hipStream_t stream) {
    hipError_t e = hipSuccess;
    // of the chunks at most one partly filled per tile beside the full ones; the
    // kernel deals them out in eight runs
    const int64_t most = std::min<int64_t>(L.ntiles, L.n / L.few) + L.n / L.part;
    if (most > 0) {
        auto kfn = k_adjoint_batch<D, kYee>;
        constexpr size_t lds = adj_lds_bytes<D>();
        e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kfn, dim3((unsigned)(8 * ((most + 7) / 8))), dim3(kAdjWG), lds,
                           stream, L.states, L.qm, L.strace, L.perm, L.tile_start,
                           L.chunk_starts, L.ntx, L.nty, L.ntiles, kAdjTile<D>, L.part, L.lam,
                           L.n, L.s_lo, L.s_hi, L.fields, pc, L.grad_fields);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if (L.few > 1) {   // (else no tile has fewer)
        auto kfn = k_adjoint_loose<D, kYee>;
        constexpr size_t lds = (kLooseWG / 64) * LaneSums<D, kYee>::kBytes;
        static_assert(lds + 8 * kLoosePart <= 80 * 1024, "two workgroups per compute unit");
        e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)lds);
        if (e != hipSuccess) return e;
        const int part = std::min(L.part, kLoosePart);
        const int64_t parts = (L.n + part - 1) / part;
        hipLaunchKernelGGL(kfn, dim3((unsigned)(8 * ((parts + 7) / 8))), dim3(kLooseWG), lds,
                           stream, L.states, L.qm, L.strace, L.perm, L.tile_start,
                           L.loose_starts, L.ntiles, part, L.lam, L.n, L.s_lo, L.s_hi, L.fields,
                           pc, L.grad_fields);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace adj
}  // namespace gcb
