// Host-side interface between the C ABI (gcb_host.hip) and the kernel
// translation units.  Each launcher enqueues its kernels on `stream` and
// returns the hipError_t of the launch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gcb_common.hpp"
#include "gcb_gr.hpp"

namespace gcb {

// Geometry of the tiled launch.
struct TileGeom {
    int tile;       // tile edge in cells
    int halo;       // extra nodes on each side of the tile in the LDS window
    int ntx, nty;   // tiles along x and y
    int window;     // tile + 2*halo nodes per side
};

// Which kernel does the work of one step.
enum class PushKind { Global, Tiled };

struct PushLaunch {
    PushKind kind;
    bool yee;              // compile-time Yee offsets
    const void* fields;    // node-interleaved device fields (double or float)
    int64_t n;
    const uint32_t* perm = nullptr;   // read slot perm[p] of the input (sort steps)
    const int32_t* tile_start;   // tiled: ntiles + 1 offsets
    TileGeom geom;
    uint8_t* trace;        // nullable: trace row of this step
    bool replay;           // read the decisions from `trace` instead of writing them
    DevStats* stats;       // nullable
    int steps = 1;         // global kernel: steps per launch (trace: steps*n bytes)
    bool exact = false;    // guiding-center branch in the exact frame (binary64 only)
    bool mirror = false;   // guiding-center branch with the mirror terms
    bool phase = false;    // guiding-center branch with the gyration phase advanced
};

// binary64 form (fields double, u double)
hipError_t launch_push_f64(const PushLaunch& L, const ParticlePtrs<double>& in,
                           const ParticlePtrs<double>& out, const PushConst& pc,
                           hipStream_t stream);

// binary64 form with contracted multiply-adds (GCB_ARITH_FAST)
hipError_t launch_push_f64_fast(const PushLaunch& L, const ParticlePtrs<double>& in,
                                const ParticlePtrs<double>& out, const PushConst& pc,
                                hipStream_t stream);

// mixed form (fields float, u float)
hipError_t launch_push_mixed(const PushLaunch& L, const ParticlePtrs<float>& in,
                             const ParticlePtrs<float>& out, const PushConst& pc,
                             hipStream_t stream);

// LDS bytes the tiled kernel needs for a window of `window` nodes per side
// (window <= kTiledMaxWindow).
size_t tiled_lds_bytes(int window, size_t elem_bytes);
constexpr int kTiledChunk = 512;       // particles a tiled workgroup queues in LDS at once
constexpr int kTiledMaxWindow = 64;    // window edge the tiled kernel stages
constexpr int kTiledMaxSteps = 16;     // steps per tiled launch (not past the next sort)
constexpr int kQueueMax = 2048;   // particles compacted per pass in a 3D tile

// ---------------------------------------------------------------------------
// 3D push

struct TileGeom3 {
    int tile;            // cubic tile edge in cells
    int halo;            // extra nodes on each side of the tile in the LDS window
    int ntx, nty, ntz;   // tiles along x, y, z
    int window;          // tile + 2*halo nodes per side
};

struct Push3Launch {
    PushKind kind;
    bool yee;              // compile-time 3D Yee offsets
    const void* fields;    // node-interleaved device fields (double or float)
    int64_t n;
    const uint32_t* perm = nullptr;   // read slot perm[p] of the input (sort steps)
    const int32_t* tile_start;   // tiled: ntiles + 1 offsets
    TileGeom3 geom;
    uint8_t* trace;        // nullable: trace row of the launch's first step
    bool replay;
    DevStats* stats;       // nullable
    int steps = 1;         // steps per launch (trace: steps*n bytes)
    bool exact = false;    // guiding-center branch in the exact frame (binary64 only)
    bool mirror = false;   // guiding-center branch with the mirror terms
    bool phase = false;    // guiding-center branch with the gyration phase advanced
};

hipError_t launch_push3_f64(const Push3Launch& L, const ParticlePtrs3<double>& in,
                            const ParticlePtrs3<double>& out, const PushConst3& pc,
                            hipStream_t stream);
// the same with contracted multiply-adds (GCB_ARITH_FAST)
hipError_t launch_push3_f64_fast(const Push3Launch& L, const ParticlePtrs3<double>& in,
                                 const ParticlePtrs3<double>& out, const PushConst3& pc,
                                 hipStream_t stream);
hipError_t launch_push3_mixed(const Push3Launch& L, const ParticlePtrs3<float>& in,
                              const ParticlePtrs3<float>& out, const PushConst3& pc,
                              hipStream_t stream);

// LDS bytes of the 3D tiled kernel for a window of `window` nodes per side.
size_t tiled3_lds_bytes(int window, size_t elem_bytes);

// ---------------------------------------------------------------------------
// cell sort

struct SortBuffers {
    uint32_t* keys;      // n
    uint32_t* idx;       // n
    uint32_t* keys2;     // n
    uint32_t* idx2;      // n
    uint32_t* hist;      // 256 * nblocks (+ scan workspace)
    uint32_t* scan_tmp;  // scan block sums
    int32_t* tile_start; // ntiles + 1
};

int64_t sort_hist_elems(int64_t n);   // elements of `hist`
int64_t sort_scan_tmp_elems(int64_t n_scan);

// Compute tile keys from positions, sort (stable), produce tile_start and the
// permutation idx (sorted slot -> source slot).
hipError_t launch_cell_sort(const double* x, const double* y, int64_t n, double inv_dx,
                            double inv_dy, const TileGeom& g, const SortBuffers& b,
                            hipStream_t stream);

// The same for the 3D state: keys are the cubic tiles of (x, y, z), row-major
// (x fastest).
hipError_t launch_cell_sort3(const double* x, const double* y, const double* z, int64_t n,
                             double inv_dx, double inv_dy, double inv_dz, const TileGeom3& g,
                             const SortBuffers& b, hipStream_t stream);

// ---------------------------------------------------------------------------
// fields

hipError_t launch_interleave_fields(const double* const comps[6], int nx, int ny,
                                    void* dst, bool to_float, hipStream_t stream);

// ---------------------------------------------------------------------------
// reductions

hipError_t launch_kinetic_energy(const void* ux, const void* uy, const void* uz,
                                 bool u_float, int64_t n, double c, double* out,
                                 double* lam_x, double* lam_y, double* lam_z,
                                 double* partial, hipStream_t stream);
int64_t kinetic_partial_elems(int64_t n);

hipError_t launch_count_flagged(const uint8_t* status, int64_t n,
                                unsigned long long* out, hipStream_t stream);

// Copies of whole arrays, all in one launch (no overlaps).  A list that is given
// more than it holds is refused by the launch.
struct CopyList {
    static constexpr int kMax = 12;   // the 3D state with q/m and ids
    void* dst[kMax];
    const void* src[kMax];
    int64_t bytes[kMax];
    int n = 0;
    bool over = false;
    void add(void* d, const void* s, int64_t b) {
        if (!s || b <= 0) return;
        if (n == kMax) {
            over = true;
            return;
        }
        dst[n] = d;
        src[n] = s;
        bytes[n++] = b;
    }
};
hipError_t launch_copy_arrays(const CopyList& L, hipStream_t stream);

// dst[s] = src[perm[s]] (inverse: dst[perm[s]] = src[s]) for n binary64 values
// of each array of a list
struct PermuteList {
    static constexpr int kMax = 10;
    const double* src[kMax];
    double* dst[kMax];
    int n = 0;
    bool over = false;
    void add(const double* s, double* d) {
        if (n == kMax) {
            over = true;
            return;
        }
        src[n] = s;
        dst[n++] = d;
    }
};
hipError_t launch_permute(const PermuteList& L, const uint32_t* perm, int64_t n, bool inverse,
                          hipStream_t stream);

// zero `words` 8-byte words at p (8-byte aligned) with a kernel
hipError_t launch_zero_words(void* p, int64_t words, hipStream_t stream);

// the library's binary64 sin and cos of n values (device arrays)
hipError_t launch_sincos(const double* x, double* s, double* c, int64_t n,
                         hipStream_t stream);

// ---------------------------------------------------------------------------
// adjoint

// Reverse sweep: threads and most particles of a workgroup, and the edges of
// its LDS window (nodes) and of its tile (cells) in 2D and 3D.
constexpr int kAdjWG = 512;
constexpr int kAdjPart = 2048;
template <int D>
constexpr int kAdjWindow = D == 2 ? 40 : 11;
template <int D>
constexpr int kAdjTile = D == 2 ? 32 : 6;
// Threads and most particles of a workgroup that takes those of tiles with few.
constexpr int kLooseWG = 256;
constexpr int kLoosePart = 1024;
template <int D>
constexpr size_t adj_lds_bytes() {
    return (size_t)6 * kAdjWindow<D> * kAdjWindow<D> * (D == 3 ? kAdjWindow<D> : 1) *
               2 * sizeof(double) + kAdjPart * sizeof(uint16_t);
}
static_assert(adj_lds_bytes<2>() + 1024 <= 160 * 1024 && adj_lds_bytes<3>() + 1024 <= 160 * 1024,
              "the window of the reverse sweep has to fit in LDS");

// One batch of the reverse sweep: the steps [s_lo, s_hi) of a segment.
struct AdjointLaunch {
    bool yee;
    const double* fields;         // node-interleaved binary64
    int64_t n;
    const double* states;         // the segment's start states, step by step (7 or 9 arrays of n)
    const double* qm;             // nullable
    const uint8_t* strace;        // the segment's decisions, step by step (1 = Boris)
    const uint32_t* perm;         // cell sort of the particles: slot -> particle
    const int32_t* tile_start;    // its tiles (ntx x nty (x ntz), kAdjTile cells)
    int ntx, nty, ntiles;
    int part;                     // particles per chunk, at most kAdjPart
    int few;                      // particles below which a tile gets no chunk
    const int32_t* chunk_starts;  // launch_chunk_starts
    const int32_t* loose_starts;
    double* lam;                  // 7 or 9 arrays of n: cotangents, in place
    int s_lo, s_hi;
    double* grad_fields;          // node-interleaved gradient accumulators
};

// starts[t], loose[t] (ntiles + 1 each): in the tiles before t, the chunks of
// `part` particles of those with at least `few`, the particles of the others
// (sums: chunk_sums_elems of scratch)
int64_t chunk_sums_elems(int ntiles);
hipError_t launch_chunk_starts(const int32_t* tile_start, int ntiles, int part, int few,
                               int32_t* starts, int32_t* loose, uint64_t* sums,
                               hipStream_t stream);
hipError_t launch_adjoint_batch(const AdjointLaunch& L, const PushConst& pc, hipStream_t stream);
hipError_t launch_adjoint3_batch(const AdjointLaunch& L, const PushConst3& pc,
                                 hipStream_t stream);

hipError_t launch_deinterleave_add(const double* grad_fields, int nx, int ny,
                                   float* const out[6], hipStream_t stream);

// curved-spacetime push (gcb_gr.hip)
struct GrPtrs {
    double *r, *th, *ph;
    void *ur, *uth, *uph;   // double (binary64 form) or float (precision form)
    const double* qm;       // nullable
    int32_t* id;            // nullable
    uint8_t* status;
};

// stable sort of the particles by (r, theta) tiles of tile x tile cells;
// the permutation ends in b.idx
hipError_t launch_gr_cell_sort(const double* r, const double* th, int64_t n,
                               const gr::GrConst& g, int tile, const SortBuffers& b,
                               hipStream_t stream);

hipError_t launch_gr_cell_lengths(const gr::GrConst& g, double dr, double dth, double* dl,
                                  hipStream_t stream);
// n_steps steps; the first launch reads slot perm[k] of `in` (k when perm is
// null) and writes slot k of `out`, later ones work in place on `out`;
// trace[step*n + (id ? id : slot)]
hipError_t launch_gr_push_f64(const GrPtrs& in, const GrPtrs& out, const uint32_t* perm,
                              int64_t n, int n_steps, const double* F, const double* dl,
                              const gr::GrConst& g, uint8_t* trace, int trace_step0,
                              DevStats* stats, hipStream_t stream);
hipError_t launch_gr_push_mixed(const GrPtrs& in, const GrPtrs& out, const uint32_t* perm,
                                int64_t n, int n_steps, const float* F, const double* dl,
                                const gr::GrConst& g, uint8_t* trace, int trace_step0,
                                DevStats* stats, hipStream_t stream);
hipError_t launch_gr_push_fast(const GrPtrs& in, const GrPtrs& out, const uint32_t* perm,
                               int64_t n, int n_steps, const double* F, const double* dl,
                               const gr::GrConst& g, uint8_t* trace, int trace_step0,
                               DevStats* stats, hipStream_t stream);

}  // namespace gcb
