// Definitions shared by the device code and the host launchers of libgcb.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// Per-particle arithmetic is compiled for the device and, for host-side
// checks of the same code, for the host.
#define GCB_HD __host__ __device__ __forceinline__

namespace gcb {

enum : uint32_t {
    ST_NONFINITE = 1,
    ST_KAPPA = 2,
    ST_QUAD = 4,
    ST_BZERO = 8,
    ST_FPRES = 16,
    ST_HALO = 32,
    ST_MIRROR = 128,
};

// Gyration handling of a guiding-center step (the values of
// gcb_params.gyration): mu conserved, u_perp_g held, mu = 0, mu conserved
// with the gyration phase advanced over the step.
enum : int32_t {
    GYR_MU = 0,
    GYR_UPERP = 1,
    GYR_ZERO = 2,
    GYR_PHASE = 3,
};

// Variants of the guiding-center branch, one kernel instance each: the
// paper's reduced frame, the exact frame of Sec. 2.2 with the zero-curvature
// scheme, the reduced frame with the mirror force and grad-B drift
// (gcb_params.frame and .mirror), the reduced frame with the gyration phase
// advanced (GYR_PHASE), and the exact frame with the curvature scheme.
enum : int {
    kVarReduced = 0,
    kVarExact = 1,
    kVarMirror = 2,
    kVarPhase = 3,
    kVarExactCurv = 4,
};

// the exact frame (either scheme)
constexpr bool var_exact(int v) { return v == kVarExact || v == kVarExactCurv; }

// 1 - v_E^2/c^2 is clamped to this floor where the drift reaches c.
constexpr double kKappaFloor = 1.0e-12;
// |1 - (dt/2) v_E.(b.grad)b| below this: no division in the parallel update.
constexpr double kDFloor = 1.0e-12;

// Lattice coordinates (position / cell size) of magnitude this or more, or
// NaN, have no field: a gather there returns NaN (a runaway iteration).
constexpr double kFarLattice = 1073741824.0;   // 2^30

// 1/sqrt(x) for finite x > 0 in binary64: the hardware estimate (good to
// about 2^-24) refined by one third-order step, y <- y (1 + e/2 + 3 e^2/8) with
// e = 1 - x y^2: the next term of the series, 5 e^3/16, lies below 2^-68.
// Five operations where two Newton-Raphson steps took eight, with the same
// error (the rounding of e and of the last sum: within two units in the last
// place).
GCB_HD double rsqrt_nr(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rsq(x);
#else
    const double y = 1.0 / sqrt(x);
#endif
    const double e = fma(-(x * y), y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// 1/x for finite normal x in binary64: the hardware estimate refined by one
// third-order step, y <- y (1 + e + e^2) with e = 1 - x y (the next term, e^3,
// lies below 2^-68); within a unit in the last place.
GCB_HD double rcp_nr(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rcp(x);
#else
    const double y = 1.0 / x;
#endif
    const double e = fma(-x, y, 1.0);
    return fma(y, fma(e, e, e), y);
}

// The same where x may be 0 or infinite: the estimate, 1/x there, stays.
GCB_HD double rcp_nr0(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    const double y = __builtin_amdgcn_rcp(x);
#else
    const double y = 1.0 / x;
#endif
    const double e = fma(-x, y, 1.0);
    return e == e ? fma(y, fma(e, e, e), y) : y;
}

// sqrt(x) for finite x > 0 in binary64, from the refined reciprocal square root
GCB_HD double sqrt_pos(double x) {
    const double y = rsqrt_nr(x);
    const double s = x * y;
    return fma(fma(-s, s, x), 0.5 * y, s);
}

// the same for x >= 0 (0, infinity and NaN stay)
GCB_HD double sqrt_nr(double x) {
#if defined(__HIP_DEVICE_COMPILE__)
    if (__builtin_amdgcn_class(x, 0x260)) return x;   // -0, +0, +inf
#else
    if (x == 0.0 || x == __builtin_inf()) return x;
#endif
    return sqrt_pos(x);
}

// a/b for finite normal b in binary64 from the refined reciprocal: the quotient
// corrected by its own remainder (rounded as a division, up to ties)
GCB_HD double div_nr(double a, double b) {
    const double r = rcp_nr(b);
    const double q = a * r;
    return fma(fma(-b, q, a), r, q);
}

// E/B < f_E > 0 by the squares (production form; the smallest number added
// matters where the limit's square rounds to 0: E^2 is then either 0, and so
// below, or larger)
GCB_HD bool below_limit(double E2, double B, double f_E) {
    const double lim = f_E * B;
    return E2 < fma(lim, lim, 0x1p-1074);
}

// 2D Yee lattice offsets (cells) of Ex, Ey, Ez, Bx, By, Bz.
constexpr double kYeeStagger[6][2] = {
    {0.5, 0.0}, {0.0, 0.5}, {0.0, 0.0}, {0.0, 0.5}, {0.5, 0.0}, {0.5, 0.5}};

// Per-launch constants, passed by value as a kernel argument.
struct PushConst {
    double dt, c, c2, inv_c2;
    double f_rho, f_E, inv_dl, fp_tol;
    double inv_dx, inv_dy, Lx, Ly;
    double qm;               // used when the per-particle array is absent
    // the production binary64 form: 1/Lx, 1/Ly and c^2/dl
    double inv_Lx, inv_Ly, c2_inv_dl;
    double stagger[6][2];
    int32_t nx, ny;
    int32_t curvature, n_iter;
    int32_t gyration, pad_;  // GYR_*
    double mirror_tol;       // > 0: ST_MIRROR where (v_perp_g/c)^2 exceeds it
};

// Device pointers of a structure-of-arrays particle state.
template <typename U>
struct ParticlePtrs {
    double* x;
    double* y;
    double* xp;
    double* yp;
    U* ux;
    U* uy;
    U* uz;
    double* qm;      // may be null
    int32_t* id;     // may be null
    uint8_t* status;
    // binary64 push, optional: the start state of every step of a launch,
    // recorded for the adjoint (step s at rec + 7*n*s: arrays x, y, xp, yp,
    // ux, uy, uz of n doubles, a particle at its trace column)
    double* rec;
};

// 3D lattice: the constants of a 2D launch (physics, x and y geometry, the
// x and y lattice offsets in b.stagger) plus the z geometry.
struct PushConst3 {
    PushConst b;
    double inv_dz, Lz;
    double inv_Lz;           // 1/Lz (the production binary64 form)
    double sz[6];            // z offsets of the lattices, in cells
    int32_t nz, pad_;
};

// 3D state: the 2D arrays plus z and its previous value.
template <typename U>
struct ParticlePtrs3 {
    ParticlePtrs<U> b;
    double* z;
    double* zp;
};

// Accumulators filled by the push kernels when statistics are requested:
// kStatSlots copies, one cache line each; workgroup b adds to slot
// b % kStatSlots so that the atomics of a launch spread over many L2 lines,
// and the host sums the slots.
constexpr int kStatSlots = 512;
struct alignas(64) DevStats {
    unsigned long long gca_steps;
    unsigned long long boris_steps;
    unsigned long long halo_misses;
    unsigned long long max_res_bits;   // bit pattern of a non-negative double
};

GCB_HD int wrap_index(int i, int n) {
    if ((unsigned)i < (unsigned)n) return i;
    int r = i % n;
    return r < 0 ? r + n : r;
}

}  // namespace gcb
