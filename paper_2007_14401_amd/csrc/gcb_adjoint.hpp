// Reverse-mode derivative (vector-Jacobian products) of one binary64 step of
// the coupled pusher in D = 2 or 3 dimensions, with the switch decision held at
// its forward value.
//
// The forward values come from the production arithmetic of gcb_math.hpp (the
// states and decisions they are evaluated at are the forward pass's own).
// Every building block has a hand-written adjoint, and a block's adjoint takes
// the forward values it needs from its inputs.  Cotangents are accumulated (+=).
//   sample_at        the six components at a point with all first derivatives
//                    and the mixed second ones of B (everything the reverse
//                    sweep needs of the fields, from one gather)
//   point_back       cotangents of E, B and of the B gradients -> node
//                    cotangents (to a window, see gcb_adjoint_kernels.hpp) and
//                    the position cotangent, including the mixed second
//                    derivatives of W carried by the gradient cotangents
//   local_back       b, v_E, kappa, E_par
//   gamma_back       Gamma(R, u_par) (eq. lfacgca2) and 1/Gamma
//   vcurv_back       curvature drift (eq. curvdrift)
//   scalars_back     A = v_E.(b.grad)b, C = v_E.(v_E.grad)b
//   drift_back       u_par b/Gamma + v_E + v_c
//   parallel_back    the parallel update (Sec. 2.2.2) through the root of the
//                    quadratic by the implicit-function derivative
//                    dG = -(G^2 dk1 + G dk2 + dk3)/(2 k1 G + k2)
//   boris_vjp        relativistic Boris push and position update
//   gca_vjp          the guiding-center step (Sec. 3.1): decomposition,
//                    parallel update, K fixed-point iterations (reversed in
//                    order), reconstruction
// State order: positions, previous positions, u (2 D + 3 values).
#pragma once

#include "gcb_math3.hpp"

namespace gcb {
namespace adj {

using LocalD = Local<double>;

// what differs between two and three dimensions
template <int D>
struct Dim;

template <>
struct Dim<2> {
    using Push = PushConst;
    using Const = Consts<double>;
    using Acc = TileAcc<double>;
    using Direct = GlobalAcc<double>;
    using Smp = Sample<double>;
    GCB_HD static const PushConst& base(const Push& pc) { return pc; }
    GCB_HD static Const consts(const Push& pc) { return make_consts<double>(pc); }
    GCB_HD static Acc acc(const double* lds, const double* F, const Push& pc, const int o[2],
                          int W) {
        return Acc{lds, F, pc.nx, pc.ny, o[0], o[1], W, false};
    }
    GCB_HD static Direct direct(const double* F, const Push& pc) {
        return Direct{F, pc.nx, pc.ny};
    }
    GCB_HD static double inv_d(const Push& pc, int a) { return a == 0 ? pc.inv_dx : pc.inv_dy; }
    GCB_HD static double box(const Push& pc, int a) { return a == 0 ? pc.Lx : pc.Ly; }
    GCB_HD static double inv_box(const Push& pc, int a) {
        return a == 0 ? pc.inv_Lx : pc.inv_Ly;
    }
    GCB_HD static int nodes(const Push& pc, int a) { return a == 0 ? pc.nx : pc.ny; }
    GCB_HD static double stagger(const Push& pc, int k, int a) { return pc.stagger[k][a]; }
    GCB_HD static constexpr int set(int k) { return kYeeSet[k]; }
    // set(k) in the three bits from 3 k
    GCB_HD static constexpr unsigned packed_sets() {
        return set(0) | set(1) << 3 | set(2) << 6 | set(3) << 9 | set(4) << 12 | set(5) << 15;
    }
    template <bool kYee, class A>
    GCB_HD static void gather(const A& acc, const Push& pc, const Const& K, const double X[2],
                              Smp& s) {
        gcb::gather<double, true, kYee>(acc, pc, K, X[0], X[1], s);
    }
    // gradient of the sample along axis a (per cell)
    GCB_HD static const double* grad(const Smp& s, int a) { return a == 0 ? s.dBx : s.dBy; }
};

template <>
struct Dim<3> {
    using Push = PushConst3;
    using Const = Consts3<double>;
    using Acc = TileAcc3<double>;
    using Direct = GlobalAcc3<double>;
    using Smp = Sample3<double>;
    GCB_HD static const PushConst& base(const Push& pc) { return pc.b; }
    GCB_HD static Const consts(const Push& pc) { return make_consts3<double>(pc); }
    GCB_HD static Acc acc(const double* lds, const double* F, const Push& pc, const int o[3],
                          int W) {
        return Acc{lds, GlobalAcc3<double>{F, pc.b.nx, pc.b.ny, pc.nz}, o[0], o[1], o[2], W,
                   false};
    }
    GCB_HD static Direct direct(const double* F, const Push& pc) {
        return Direct{F, pc.b.nx, pc.b.ny, pc.nz};
    }
    GCB_HD static double inv_d(const Push& pc, int a) {
        return a == 0 ? pc.b.inv_dx : a == 1 ? pc.b.inv_dy : pc.inv_dz;
    }
    GCB_HD static double box(const Push& pc, int a) {
        return a == 0 ? pc.b.Lx : a == 1 ? pc.b.Ly : pc.Lz;
    }
    GCB_HD static double inv_box(const Push& pc, int a) {
        return a == 0 ? pc.b.inv_Lx : a == 1 ? pc.b.inv_Ly : pc.inv_Lz;
    }
    GCB_HD static int nodes(const Push& pc, int a) {
        return a == 0 ? pc.b.nx : a == 1 ? pc.b.ny : pc.nz;
    }
    GCB_HD static double stagger(const Push& pc, int k, int a) {
        return a < 2 ? pc.b.stagger[k][a] : pc.sz[k];
    }
    GCB_HD static constexpr int set(int k) { return kYee3Set[k]; }
    GCB_HD static constexpr unsigned packed_sets() {
        return set(0) | set(1) << 3 | set(2) << 6 | set(3) << 9 | set(4) << 12 | set(5) << 15;
    }
    template <bool kYee, class A>
    GCB_HD static void gather(const A& acc, const Push& pc, const Const& K, const double X[3],
                              Smp& s) {
        gcb::gather3<double, true, kYee>(acc, pc, K, X[0], X[1], X[2], s);
    }
    GCB_HD static const double* grad(const Smp& s, int a) {
        return a == 0 ? s.dBx : a == 1 ? s.dBy : s.dBz;
    }
};

// ---------------------------------------------------------------------------
// gather

// A gather point of the reverse sweep: the values, their derivatives along each
// axis (per cell), the mixed second derivatives of B, the weights per axis (on
// the Yee lattice one per offset 0 or 1/2, else one per component) and the
// nodes (0, 0(, 0)) of the six stencils in the window, if all lie inside.
template <int D, bool kYee>
struct Point {
    static constexpr int kSets = kYee ? 2 : 6;
    double v[6];
    double d[D][6];
    double m[D * (D - 1) / 2][3];   // xy (xz, yz) of B
    double w[D][kSets];
    int off[6];
    bool in;
    bool far;   // a runaway point: its sample is a constant NaN

    // the entry of component k along axis a
    GCB_HD static constexpr int entry(int k, int a) {
        return kYee ? (Dim<D>::set(k) >> a) & 1 : k;
    }
};

template <bool kYee>
GCB_HD void eval_point(int k, double f00, double f10, double f01, double f11,
                       Point<2, kYee>& p) {
    const double wx = p.w[0][p.entry(k, 0)], wy = p.w[1][p.entry(k, 1)];
    double c[4];
    cell_coefs(f00, f10, f01, f11, c);
    eval_coefs<true>(c, wx, wy, p.v[k], p.d[0][k], p.d[1][k]);
    if (k >= 3) p.m[0][k - 3] = c[3];
}

template <bool kYee>
GCB_HD void eval_point(int k, const double f[8], Point<3, kYee>& p) {
    const double wx = p.w[0][p.entry(k, 0)], wy = p.w[1][p.entry(k, 1)],
                 wz = p.w[2][p.entry(k, 2)];
    double d[4], e[4];   // along x at (y, z) = (0,0), (1,0), (0,1), (1,1)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        d[i] = f[2 * i + 1] - f[2 * i];
        e[i] = f[2 * i] + wx * d[i];
    }
    const double y0 = e[1] - e[0], y1 = e[3] - e[2];
    const double v0 = e[0] + wy * y0;
    const double dz = (e[2] + wy * y1) - v0;
    const double q0 = d[1] - d[0], q1 = d[3] - d[2];
    const double x0 = d[0] + wy * q0, x1 = d[2] + wy * q1;
    p.v[k] = v0 + wz * dz;
    p.d[0][k] = x0 + wz * (x1 - x0);
    p.d[1][k] = y0 + wz * (y1 - y0);
    p.d[2][k] = dz;
    if (k >= 3) {
        p.m[0][k - 3] = q0 + wz * (q1 - q0);
        p.m[1][k - 3] = x1 - x0;
        p.m[2][k - 3] = y1 - y0;
    }
}

// cells c and weights of the point X
template <int D, bool kYee>
GCB_HD void place(const typename Dim<D>::Push& pc, const double X[D],
                  int c[D][Point<D, kYee>::kSets], Point<D, kYee>& p) {
    double g[D];
    p.far = false;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        g[a] = X[a] * Dim<D>::inv_d(pc, a);
        p.far = p.far || !(fabs(g[a]) < kFarLattice);
    }
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const double ga = p.far ? 0.0 : g[a];
#pragma unroll
        for (int s = 0; s < Point<D, kYee>::kSets; ++s) {
            const double xi = ga - (kYee ? 0.5 * s : Dim<D>::stagger(pc, s, a));
            const double f = floor(xi);
            c[a][s] = (int)f;
            p.w[a][s] = xi - f;
        }
    }
}

// the stencil offsets in the window (or its periodic images) of cells c
template <int D, bool kYee>
GCB_HD void locate(const typename Dim<D>::Push& pc, const int o[D], int W,
                   const int c[D][Point<D, kYee>::kSets], Point<D, kYee>& p) {
    int d[D][Point<D, kYee>::kSets];
    p.in = true;
#pragma unroll
    for (int a = 0; a < D; ++a)
#pragma unroll
        for (int s = 0; s < Point<D, kYee>::kSets; ++s) {
            int i = c[a][s] - o[a];
            if ((unsigned)i > (unsigned)(W - 2)) i += i < 0 ? Dim<D>::nodes(pc, a)
                                                            : -Dim<D>::nodes(pc, a);
            p.in = p.in && (unsigned)i <= (unsigned)(W - 2);
            d[a][s] = i;
        }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        int e = 0;
#pragma unroll
        for (int a = D - 1; a >= 0; --a) e = e * W + d[a][p.entry(k, a)];
        p.off[k] = e;
    }
}

// the sample of cells c from the field array
template <bool kYee>
GCB_HD void from_grid(const GlobalAcc<double>& g, const int c[2][Point<2, kYee>::kSets],
                      Point<2, kYee>& p) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        double f00, f10, f01, f11;
        g.quad(k, c[0][p.entry(k, 0)], c[1][p.entry(k, 1)], f00, f10, f01, f11);
        eval_point(k, f00, f10, f01, f11, p);
    }
}

template <bool kYee>
GCB_HD void from_grid(const GlobalAcc3<double>& g, const int c[3][Point<3, kYee>::kSets],
                      Point<3, kYee>& p) {
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        double f[8];
        g.oct<double>(k, c[0][p.entry(k, 0)], c[1][p.entry(k, 1)], c[2][p.entry(k, 2)], f);
        eval_point(k, f, p);
    }
}

template <bool kYee>
GCB_HD void sample_at(const TileAcc<double>& acc, const PushConst& pc, const double X[2],
                      Point<2, kYee>& p) {
    int c[2][Point<2, kYee>::kSets];
    place<2>(pc, X, c, p);
    const int o[2] = {acc.oi, acc.oj}, W = acc.W;
    locate<2>(pc, o, W, c, p);
    if (__builtin_expect(p.in, 1)) {
        const int set[4] = {p.off[2], p.off[0], p.off[1], p.off[5]};
        const LdsLoad<double> ld{acc.lds, set, W, W * W};
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            double f00, f10, f01, f11;
            if constexpr (kYee) {
                ld.load4<double>(kYeeSet[k], k, f00, f10, f01, f11);
            } else {
                const double* q = acc.lds + window_elem<double>(k, p.off[k], W * W);
                const int st = window_step<double>(k);
                f00 = q[0];
                f10 = q[st];
                f01 = q[st * W];
                f11 = q[st * (W + 1)];
            }
            eval_point(k, f00, f10, f01, f11, p);
        }
    } else {
        from_grid(GlobalAcc<double>{acc.F, acc.nx, acc.ny}, c, p);
    }
}

template <bool kYee>
GCB_HD void sample_at(const TileAcc3<double>& acc, const PushConst3& pc, const double X[3],
                      Point<3, kYee>& p) {
    int c[3][Point<3, kYee>::kSets];
    place<3>(pc, X, c, p);
    const int o[3] = {acc.oi, acc.oj, acc.ol}, W = acc.W;
    locate<3>(pc, o, W, c, p);
    if (__builtin_expect(p.in, 1)) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            double f[8];
            const LdsLoad3<double> ld{acc.lds, &p.off[k], W, W * W, W * W * W};
            ld.load8<double>(0, k, f);
            eval_point(k, f, p);
        }
    } else {
        from_grid(acc.g, c, p);
    }
}

template <bool kYee>
GCB_HD void sample_at(const GlobalAcc<double>& acc, const PushConst& pc, const double X[2],
                      Point<2, kYee>& p) {
    int c[2][Point<2, kYee>::kSets];
    place<2>(pc, X, c, p);
    from_grid(acc, c, p);
}

template <bool kYee>
GCB_HD void sample_at(const GlobalAcc3<double>& acc, const PushConst3& pc, const double X[3],
                      Point<3, kYee>& p) {
    int c[3][Point<3, kYee>::kSets];
    place<3>(pc, X, c, p);
    from_grid(acc, c, p);
}

// The point as the sample that the forward functions take (a runaway point's
// is NaN, as the gather has it).
template <bool kYee>
GCB_HD void to_sample(const Point<2, kYee>& p, Sample<double>& s) {
    const double nan = __builtin_nan("");
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        s.E[i] = p.far ? nan : p.v[i];
        s.B[i] = p.far ? nan : p.v[3 + i];
        s.dBx[i] = p.far ? nan : p.d[0][3 + i];
        s.dBy[i] = p.far ? nan : p.d[1][3 + i];
    }
}

template <bool kYee>
GCB_HD void to_sample(const Point<3, kYee>& p, Sample3<double>& s) {
    const double nan = __builtin_nan("");
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        s.E[i] = p.far ? nan : p.v[i];
        s.B[i] = p.far ? nan : p.v[3 + i];
        s.dBx[i] = p.far ? nan : p.d[0][3 + i];
        s.dBy[i] = p.far ? nan : p.d[1][3 + i];
        s.dBz[i] = p.far ? nan : p.d[2][3 + i];
    }
}

// Cotangents of E, B and of the B gradients per cell at a point.
template <int D>
struct SampleBar {
    double v[6];      // E, B
    double g[D][3];   // d_a B

    GCB_HD SampleBar() {
#pragma unroll
        for (int k = 0; k < 6; ++k) v[k] = 0.0;
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int i = 0; i < 3; ++i) g[a][i] = 0.0;
    }
};

// The four node cotangents of a bilinear cell from those of the value and of
// the two gradients: the transpose of cell_coefs and eval_coefs.
GCB_HD void plane_back(double vb, double gx, double gy, double wx, double wy, double o[4]) {
    const double cx = vb * wx + gx;
    const double cy = vb * wy + gy;
    const double cxy = wy * cx + gy * wx;
    o[3] = cxy;
    o[1] = cx - cxy;
    o[2] = cy - cxy;
    o[0] = (vb - cx) - o[2];
}

// Node cotangents of component k (2^D values, x fastest).
template <bool kYee>
GCB_HD void nodes_back(const Point<2, kYee>& p, const SampleBar<2>& sb, int k, double o[4]) {
    plane_back(sb.v[k], k < 3 ? 0.0 : sb.g[0][k - 3], k < 3 ? 0.0 : sb.g[1][k - 3],
               p.w[0][p.entry(k, 0)], p.w[1][p.entry(k, 1)], o);
}

template <bool kYee>
GCB_HD void nodes_back(const Point<3, kYee>& p, const SampleBar<3>& sb, int k, double o[8]) {
    const double wx = p.w[0][p.entry(k, 0)], wy = p.w[1][p.entry(k, 1)],
                 wz = p.w[2][p.entry(k, 2)], az = 1.0 - wz;
    if (k < 3) {
        plane_back(sb.v[k] * az, 0.0, 0.0, wx, wy, o);
        plane_back(sb.v[k] * wz, 0.0, 0.0, wx, wy, o + 4);
    } else {
        const double v = sb.v[k], gx = sb.g[0][k - 3], gy = sb.g[1][k - 3], gz = sb.g[2][k - 3];
        plane_back(v * az - gz, gx * az, gy * az, wx, wy, o);
        plane_back(v * wz + gz, gx * wz, gy * wz, wx, wy, o + 4);
    }
}

// index of the mixed derivative along axes a and b
GCB_HD constexpr int mixed(int a, int b) { return a + b - 1; }   // xy 0, xz 1, yz 2

// Cotangents of the sample at X to the nodes (by `win`) and to the position.
template <int D, bool kYee, class Win>
GCB_HD void point_back(const Win& win, const typename Dim<D>::Push& pc, const double X[D],
                       const Point<D, kYee>& p, const SampleBar<D>& sb, double Xb[D]) {
    // a runaway point's sample is a constant NaN: it depends on nothing
    if (p.far) return;
    win.add(pc, X, p, sb);
#pragma unroll
    for (int a = 0; a < D; ++a) {
        double q = 0.0;
#pragma unroll
        for (int k = 0; k < 6; ++k) q += sb.v[k] * p.d[a][k];
#pragma unroll
        for (int b = 0; b < D; ++b)
            if (b != a) {
#pragma unroll
                for (int i = 0; i < 3; ++i) q += sb.g[b][i] * p.m[mixed(a, b)][i];
            }
        Xb[a] += q * Dim<D>::inv_d(pc, a);
    }
}

// ---------------------------------------------------------------------------
// local quantities

GCB_HD double dot3(const double a[3], const double b[3]) {
    return (a[0] * b[0] + a[1] * b[1]) + a[2] * b[2];
}
GCB_HD void cross3(const double a[3], const double b[3], double c[3]) {
    c[0] = a[1] * b[2] - a[2] * b[1];
    c[1] = a[2] * b[0] - a[0] * b[2];
    c[2] = a[0] * b[1] - a[1] * b[0];
}

struct LocalBar {
    double B = 0.0, inv_B = 0.0, kappa = 0.0, Epar = 0.0;
    double b[3] = {0.0, 0.0, 0.0}, vE[3] = {0.0, 0.0, 0.0};
};

// E and B cotangents from those of b, v_E, kappa, E_par, B and 1/B.
template <int D, class S, class KC>
GCB_HD void local_back(const S& s, const LocalD& L, const KC& K, const LocalBar& Lb,
                       SampleBar<D>& sb) {
    if (L.B == 0.0) {   // b, v_E and the curvature terms are held at 0 there
        sb = SampleBar<D>();
        return;
    }
    double vEb[3], bb[3], X[3], Xb[3], t[3];
    // the clamp holds kappa: no way through it
    const double omb = L.om > kKappaFloor
                           ? (-0.5 * Lb.kappa) * ((L.kappa * L.kappa) * L.kappa) : 0.0;
    const double q = (-2.0 * K.inv_c2) * omb;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        sb.v[i] += Lb.Epar * L.b[i];
        bb[i] = Lb.b[i] + Lb.Epar * s.E[i];
        vEb[i] = Lb.vE[i] + q * L.vE[i];
    }
    cross3(s.E, s.B, X);
    const double sc = K.c * (L.inv_B * L.inv_B);
    const double scb = dot3(vEb, X);
#pragma unroll
    for (int i = 0; i < 3; ++i) Xb[i] = sc * vEb[i];
    cross3(s.B, Xb, t);
#pragma unroll
    for (int i = 0; i < 3; ++i) sb.v[i] += t[i];
    cross3(Xb, s.E, t);
    const double invBb = (Lb.inv_B + scb * ((2.0 * K.c) * L.inv_B)) + dot3(bb, s.B);
    const double Bmb = Lb.B - invBb * (L.inv_B * L.inv_B);
#pragma unroll
    for (int i = 0; i < 3; ++i) sb.v[3 + i] += (t[i] + bb[i] * L.inv_B) + Bmb * L.b[i];
}

// ---------------------------------------------------------------------------
// Gamma, curvature drift, drift terms

// the gyration state of the differentiated step: mu conserved (the adjoint
// serves the paper's eq. dmudt only)
GCB_HD Gyr<double> conserved_mu(double mu) { return Gyr<double>{mu, 0.0, false}; }

// Gb: cotangent of Gamma
template <class KC>
GCB_HD void gamma_back(const LocalD& L, double upar, double mu, const KC& K, double Gb,
                       LocalBar& Lb, double& uparb, double& mub) {
    const double bk = L.B * L.kappa;
    const double arg = 1.0 + (upar * upar + (2.0 * mu) * bk) * K.inv_c2;
    const double rs = rsqrt_nr(arg);
    Lb.kappa += Gb * (arg * rs);
    const double q = ((Gb * L.kappa) * rs) * K.inv_c2;   // 2 d(u_par^2 + u_perp^2)
    uparb += q * upar;
    mub += q * bk;
    Lb.B += (q * mu) * L.kappa;
    Lb.kappa += (q * mu) * L.B;
}

// igb: cotangent of 1/Gamma (inv_gam)
template <int D, class S, class KC>
GCB_HD void vcurv_back(const S& s, const LocalD& L, const typename Dim<D>::Push& pc,
                       double upar, double inv_gam, double inv_qm, const KC& K,
                       const double vcb[3], LocalBar& Lb, SampleBar<D>& sb, double& uparb,
                       double& igb) {
    const double u2 = upar * upar;
    const double a1 = u2 * inv_gam;
    double V[D], w[3] = {0.0, 0.0, 0.0}, z[3], zb[3], wb[3], t[3];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        V[a] = (a1 * L.b[a] + upar * L.vE[a]) * Dim<D>::inv_d(pc, a);
        const double* g = Dim<D>::grad(s, a);
#pragma unroll
        for (int i = 0; i < 3; ++i) w[i] += V[a] * g[i];
    }
    cross3(L.b, w, z);
    const double ci = K.c * inv_qm;
    const double kb = L.kappa * L.inv_B;
    const double pre = (kb * kb) * ci;
    const double q = (2.0 * dot3(vcb, z)) * (kb * ci);
    Lb.kappa += q * L.inv_B;
    Lb.inv_B += q * L.kappa;
#pragma unroll
    for (int i = 0; i < 3; ++i) zb[i] = pre * vcb[i];
    cross3(w, zb, t);
    cross3(zb, L.b, wb);
#pragma unroll
    for (int i = 0; i < 3; ++i) Lb.b[i] += t[i];
    double a1b = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const double* g = Dim<D>::grad(s, a);
#pragma unroll
        for (int i = 0; i < 3; ++i) sb.g[a][i] += V[a] * wb[i];
        const double Vb = dot3(g, wb) * Dim<D>::inv_d(pc, a);
        a1b += Vb * L.b[a];
        Lb.b[a] += a1 * Vb;
        uparb += Vb * L.vE[a];
        Lb.vE[a] += upar * Vb;
    }
    uparb += (a1b * 2.0) * (upar * inv_gam);
    igb += a1b * u2;
}

// Fb: cotangents of u_par b/Gamma + v_E + v_c
template <int D, class S, class KC>
GCB_HD void drift_back(const S& s, const LocalD& L, const typename Dim<D>::Push& pc,
                       double upn, double mu, double inv_qm, bool curv, const KC& K,
                       const double Fb[D], LocalBar& Lb, SampleBar<D>& sb, double& upnb,
                       double& mub) {
    const Gam<double> G = gamma_gca2(L, upn, conserved_mu(mu), K);
    const double a = upn * G.inv;
    double ab = 0.0;
#pragma unroll
    for (int i = 0; i < D; ++i) {
        ab += Fb[i] * L.b[i];
        Lb.b[i] += a * Fb[i];
        Lb.vE[i] += Fb[i];
    }
    upnb += ab * G.inv;
    double igb = ab * upn;
    if (curv) {
        const double vcb[3] = {Fb[0], Fb[1], D == 3 ? Fb[D - 1] : 0.0};
        vcurv_back<D>(s, L, pc, upn, G.inv, inv_qm, K, vcb, Lb, sb, upnb, igb);
    }
    gamma_back(L, upn, mu, K, -igb * (G.inv * G.inv), Lb, upnb, mub);
}

// u_par b/Gamma + v_E + v_c, the D components
template <int D, class S, class KC>
GCB_HD void drift_of(const S& s, const LocalD& L, double upn, double mu, double inv_qm,
                     bool curv, const KC& K, double F[D]) {
    const Gam<double> G = gamma_gca2(L, upn, conserved_mu(mu), K);
    const double a = upn * G.inv;
    double vc[3] = {0.0, 0.0, 0.0};
    if (curv) v_curv_dir(L, s, upn, G.inv, inv_qm, K, vc);
#pragma unroll
    for (int i = 0; i < D; ++i) F[i] = (a * L.b[i] + L.vE[i]) + vc[i];
}

// ---------------------------------------------------------------------------
// parallel update

// A and C (curvature_scalars_dir) from their cotangents
template <int D, class S, class KC>
GCB_HD void scalars_back(const S& s, const LocalD& L, const typename Dim<D>::Push& pc,
                         const KC& K, double Ab, double Cb, LocalBar& Lb, SampleBar<D>& sb) {
    double gb[3], gv[3], gbb[3], gvb[3];
    b_along(s, L.b, K, gb);
    b_along(s, L.vE, K, gv);
    const double Ai = Ab * L.inv_B, Ci = Cb * L.inv_B;
    Lb.inv_B += Ab * dot3(L.vE, gb) + Cb * dot3(L.vE, gv);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        Lb.vE[i] += Ai * gb[i] + Ci * gv[i];
        gbb[i] = Ai * L.vE[i];
        gvb[i] = Ci * L.vE[i];
    }
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const double id = Dim<D>::inv_d(pc, a);
        const double* g = Dim<D>::grad(s, a);
        const double ba = L.b[a] * id, va = L.vE[a] * id;
#pragma unroll
        for (int i = 0; i < 3; ++i) sb.g[a][i] += ba * gbb[i] + va * gvb[i];
        Lb.b[a] += dot3(g, gbb) * id;
        Lb.vE[a] += dot3(g, gvb) * id;
    }
}

// L holds A and C (with curv); Ab, Cb receive their cotangents
template <class KC>
GCB_HD void parallel_back(const LocalD& L, double upar, double mu, double qm, bool curv,
                          const KC& K, double upnb, LocalBar& Lb, double& uparb, double& mub,
                          double& Ab, double& Cb) {
    const double dtqm = qm * K.dt;
    Ab = Cb = 0.0;
    if (!curv) {
        uparb += upnb;
        Lb.Epar += dtqm * upnb;
        return;
    }
    const double h = K.h;
    const double A = L.A, C = L.C;
    const double G0 = gamma_gca2(L, upar, conserved_mu(mu), K).g;
    const double upr = (upar * (1.0 + h * A) + dtqm * L.Epar) + (h * G0) * C;
    const double Dd = 1.0 - h * A;
    const double DD = Dd * Dd;
    const double k1 = (h * h) * (C * C) - (K.c2 * DD) * L.om;
    const double k2 = (upr * K.dt) * C;
    const double bk = L.B * L.kappa;
    const double u2 = (2.0 * mu) * bk;
    const double k3 = upr * upr + (K.c2 + u2) * DD;
    const double disc = k2 * k2 - (4.0 * k1) * k3;
    const bool dok = fabs(Dd) >= kDFloor;
    bool ok = (k1 < 0.0) && (disc >= 0.0) && dok;
    const double sq = sqrt_nr(disc >= 0.0 ? disc : 0.0);
    const bool pos_k2 = k2 >= 0.0;
    const double num = pos_k2 ? k2 + sq : 2.0 * k3;
    double den = pos_k2 ? -2.0 * k1 : sq - k2;
    den = (ok && den > 0.0) ? den : 1.0;
    const double gp = div_nr(num, den);
    ok = ok && (gp > 0.0) && __builtin_isfinite(gp);
    if (!ok && !dok) {
        uparb += upnb;
        Lb.Epar += dtqm * upnb;
        return;
    }
    const double iD = rcp_nr(Dd);
    double uprb = upnb * iD, Db;
    const double w = uprb * h;
    if (ok) {
        const double upn = (upr + (h * gp) * C) * iD;
        const double gpb = w * C;
        Cb += w * gp;
        Db = -uprb * upn;
        const double k3b = -gpb / (2.0 * k1 * gp + k2);
        const double k2b = k3b * gp;
        const double k1b = k2b * gp;
        uprb += k3b * 2.0 * upr;
        double DDb = k3b * (K.c2 + u2);
        const double u2b = 2.0 * (k3b * DD);
        mub += u2b * bk;
        Lb.B += u2b * mu * L.kappa;
        Lb.kappa += u2b * mu * L.B;
        uprb += k2b * K.dt * C;
        Cb += k2b * upr * K.dt;
        Cb += k1b * 2.0 * (h * h) * C;
        DDb -= k1b * K.c2 * L.om;
        Lb.kappa += k1b * 2.0 * K.c2 * DD * (L.om * L.inv_kappa);
        Db += DDb * 2.0 * Dd;
    } else {
        // fallback: Gamma taken at u'/D (no implicit term)
        const double v = upr * iD;
        const double gfb = gamma_gca2(L, v, conserved_mu(mu), K).g;
        const double upn = (upr + (h * gfb) * C) * iD;
        const double gfbb = w * C;
        Cb += w * gfb;
        Db = -uprb * upn;
        double vb = 0.0;
        gamma_back(L, v, mu, K, gfbb, Lb, vb, mub);
        uprb += vb * iD;
        Db -= vb * v * iD;
    }
    Ab = h * (uprb * upar - Db);
    uparb += uprb * (1.0 + h * A);
    Lb.Epar += uprb * dtqm;
    Cb += uprb * h * G0;
    gamma_back(L, upar, mu, K, uprb * h * C, Lb, uparb, mub);
}

// ---------------------------------------------------------------------------
// steps.  st = (x, previous x, u) at the step start; lam holds the cotangents
// of the step outputs on entry and of its inputs on return.

template <int D, bool kYee, class Acc, class Win>
GCB_HD void boris_vjp(const Acc& acc, const Win& win,
                      const typename Dim<D>::Push& pc, const typename Dim<D>::Const& K,
                      const double st[2 * D + 3], double qm, double lam[2 * D + 3]) {
    Point<D, kYee> p;
    sample_at(acc, pc, st, p);
    typename Dim<D>::Smp s;
    to_sample(p, s);
    const double* u = st + 2 * D;
    double* ub = lam + 2 * D;
    const double dt = K.dt;
    // forward
    const double hq = (qm * dt) * 0.5;
    double um[3], t[3], sv[3], up[3], un[3], x[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) um[i] = u[i] + hq * s.E[i];
    // (1/Gamma is 0 where u^2 overflows: no rotation, no motion, and cotangents
    // of u that pass through)
    const double g2 = 1.0 + dot3(um, um) * K.inv_c2;
    const double igm = __builtin_isinf(g2) ? 0.0 : rsqrt_nr(g2);
    const double f = __builtin_isinf(g2) ? 0.0 : div_nr(hq, K.c * sqrt_pos(g2));   // as the push
#pragma unroll
    for (int i = 0; i < 3; ++i) t[i] = f * s.B[i];
    const double g = 2.0 * rcp_nr0(1.0 + dot3(t, t));
#pragma unroll
    for (int i = 0; i < 3; ++i) sv[i] = g * t[i];
    cross3(um, t, x);
#pragma unroll
    for (int i = 0; i < 3; ++i) up[i] = um[i] + x[i];
    cross3(up, sv, x);
#pragma unroll
    for (int i = 0; i < 3; ++i) un[i] = (um[i] + x[i]) + hq * s.E[i];
    const double gn2 = 1.0 + dot3(un, un) * K.inv_c2;
    const double ign = __builtin_isinf(gn2) ? 0.0 : rsqrt_nr(gn2);
    // reverse: x^{n+1} = x^n + dt un/Gamma
    double unb[3] = {ub[0], ub[1], ub[2]}, igb = 0.0;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        unb[a] += dt * ign * lam[a];
        igb += dt * un[a] * lam[a];
    }
    const double gnb = -igb * (ign * ign);
#pragma unroll
    for (int i = 0; i < 3; ++i) unb[i] += (gnb * K.inv_c2 * ign) * un[i];
    SampleBar<D> sb;
    double umb[3], upb[3], svb[3], tb[3];
    // un = uq + hq E, uq = um + up x s
    cross3(sv, unb, upb);
    cross3(unb, up, svb);
    // up = um + um x t
    cross3(t, upb, x);
#pragma unroll
    for (int i = 0; i < 3; ++i) umb[i] = (unb[i] + upb[i]) + x[i];
    cross3(upb, um, tb);
    // s = g t, g = 2/(1 + t^2)
    const double gb = dot3(svb, t);
    const double t2b = -gb * (g * g) * 0.5;
#pragma unroll
    for (int i = 0; i < 3; ++i) tb[i] += g * svb[i] + (2.0 * t2b) * t[i];
    // t = f B, f = hq/(c Gamma)
    const double fb = dot3(tb, s.B);
    const double gmb = -fb * f * igm;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        sb.v[3 + i] = f * tb[i];
        umb[i] += (gmb * K.inv_c2 * igm) * um[i];
        sb.v[i] = hq * (unb[i] + umb[i]);
    }
    // (x, u) of the step start; the previous position has no part in the step,
    // and x^n is the next one's previous position
    double Xb[D];
#pragma unroll
    for (int a = 0; a < D; ++a) {
        Xb[a] = lam[a] + lam[D + a];
        lam[D + a] = 0.0;
    }
    point_back<D, kYee>(win, pc, st, p, sb, Xb);
#pragma unroll
    for (int a = 0; a < D; ++a) lam[a] = Xb[a];
#pragma unroll
    for (int i = 0; i < 3; ++i) ub[i] = umb[i];
}

constexpr int kMaxAdjIter = 8;   // fixed-point iterations the adjoint supports

template <int D, bool kYee, class Acc, class Win>
GCB_HD void gca_vjp(const Acc& acc, const Win& win,
                    const typename Dim<D>::Push& pc, const typename Dim<D>::Const& K,
                    const double st[2 * D + 3], double qm, double lam[2 * D + 3]) {
    using Smp = typename Dim<D>::Smp;
    const PushConst& pb = Dim<D>::base(pc);
    const bool curv = pb.curvature != 0;
    const double* u = st + 2 * D;
    const double inv_qm = rcp_nr0(qm);
    const double h = K.h;
    const int Kit = pb.n_iter < kMaxAdjIter ? pb.n_iter : kMaxAdjIter;

    // ---- forward recomputation (values the reverse sweep needs)
    double Rh[D];
#pragma unroll
    for (int a = 0; a < D; ++a)
        Rh[a] = st[a] - 0.5 * min_image_i<double>(st[a] - st[D + a], Dim<D>::box(pc, a),
                                                  Dim<D>::inv_box(pc, a));
    double upar, mu, bp[3];
    {
        Smp s;
        LocalD L;
        Dim<D>::template gather<kYee>(acc, pc, K, Rh, s);
        local_fields(s.E, s.B, K, L);
        upar = dot3(u, L.b);
        const Gam<double> G = gamma_full2(u[0], u[1], u[2], K);
        double vc[3] = {0.0, 0.0, 0.0};
        if (curv) v_curv_dir(L, s, upar, G.inv, inv_qm, K, vc);
#pragma unroll
        for (int i = 0; i < 3; ++i) bp[i] = (u[i] - upar * L.b[i]) - (L.vE[i] + vc[i]) * G.g;
        const double up2 = dot3(bp, bp);
        mu = ((0.5 * up2) * L.inv_B) * L.inv_kappa;
        const double inv_nu = up2 > 0.0 ? rsqrt_nr(up2) : 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) bp[i] *= inv_nu;
    }
    double upn, Fn[D];
    {
        Smp s;
        LocalD L;
        Dim<D>::template gather<kYee>(acc, pc, K, st, s);
        local_fields(s.E, s.B, K, L);
        if (curv) curvature_scalars_dir(s, K, L);
        uint32_t fl = 0;
        upn = parallel_update(L, upar, conserved_mu(mu), qm, curv, K, fl);
        drift_of<D>(s, L, upn, mu, inv_qm, curv, K, Fn);
    }
    double Rk[kMaxAdjIter][D], Rx[D];   // R^1..R^{K-1}, then R^K
#pragma unroll
    for (int a = 0; a < D; ++a) Rx[a] = st[a] + h * (Fn[a] + Fn[a]);
    for (int k = 1; k < Kit; ++k) {
        Smp s;
        LocalD L;
        double F[D];
#pragma unroll
        for (int a = 0; a < D; ++a) Rk[k][a] = Rx[a];
        Dim<D>::template gather<kYee>(acc, pc, K, Rx, s);
        local_fields(s.E, s.B, K, L);
        drift_of<D>(s, L, upn, mu, inv_qm, curv, K, F);
#pragma unroll
        for (int a = 0; a < D; ++a) Rx[a] = st[a] + h * (Fn[a] + F[a]);
    }

    // ---- reverse sweep
    double xb[D], Rb[D];   // xp_out = x, x_out = wrap(R^K)
#pragma unroll
    for (int a = 0; a < D; ++a) {
        xb[a] = lam[D + a];
        Rb[a] = lam[a];
    }
    double upnb = 0.0, mub = 0.0, bpb[3];

    // 5. reconstruction at R^{n+1/2}
    {
        double Rm[D], Rmb[D];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            Rm[a] = st[a] + 0.5 * (Rx[a] - st[a]);
            Rmb[a] = 0.0;
        }
        const double* ub = lam + 2 * D;
        Point<D, kYee> p;
        Smp s;
        LocalD L;
        sample_at(acc, pc, Rm, p);
        to_sample(p, s);
        local_fields(s.E, s.B, K, L);
        LocalBar Lb;
        SampleBar<D> sb;
        const Gam<double> G = gamma_gca2(L, upn, conserved_mu(mu), K);
        double vc[3] = {0.0, 0.0, 0.0};
        if (curv) v_curv_dir(L, s, upn, G.inv, inv_qm, K, vc);
        const double bk = L.B * L.kappa;
        const double up2 = (2.0 * mu) * bk;
        const double ium = up2 > 0.0 ? rsqrt_nr(up2) : 0.0;
        const double um = up2 * ium;
        upnb += dot3(ub, L.b);
        double vcb[3], gb = 0.0, igb = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            Lb.b[i] += upn * ub[i];
            vcb[i] = G.g * ub[i];
            Lb.vE[i] += vcb[i];
            gb += (L.vE[i] + vc[i]) * ub[i];
            bpb[i] = um * ub[i];
        }
        const double q = dot3(bp, ub) * ium;   // 2 d(um^2)
        mub += q * bk;
        Lb.B += q * mu * L.kappa;
        Lb.kappa += q * mu * L.B;
        if (curv) vcurv_back<D>(s, L, pc, upn, G.inv, inv_qm, K, vcb, Lb, sb, upnb, igb);
        gamma_back(L, upn, mu, K, gb - igb * (G.inv * G.inv), Lb, upnb, mub);
        local_back<D>(s, L, K, Lb, sb);
        point_back<D, kYee>(win, pc, Rm, p, sb, Rmb);
#pragma unroll
        for (int a = 0; a < D; ++a) {
            xb[a] += 0.5 * Rmb[a];
            Rb[a] += 0.5 * Rmb[a];
        }
    }

    // 4. fixed-point iterations in reverse order
    double Fnb[D];
#pragma unroll
    for (int a = 0; a < D; ++a) Fnb[a] = 0.0;
    for (int k = Kit - 1; k >= 0; --k) {
        double Fb[D];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            xb[a] += Rb[a];
            Fb[a] = h * Rb[a];
            Fnb[a] += Fb[a];
            Rb[a] = 0.0;
        }
        if (k == 0) {
#pragma unroll
            for (int a = 0; a < D; ++a) Fnb[a] += Fb[a];
        } else {
            Point<D, kYee> p;
            Smp s;
            LocalD L;
            sample_at(acc, pc, Rk[k], p);
            to_sample(p, s);
            local_fields(s.E, s.B, K, L);
            LocalBar Lb;
            SampleBar<D> sb;
            drift_back<D>(s, L, pc, upn, mu, inv_qm, curv, K, Fb, Lb, sb, upnb, mub);
            local_back<D>(s, L, K, Lb, sb);
            point_back<D, kYee>(win, pc, Rk[k], p, sb, Rb);
        }
    }

    // 3.-2. drift at R^n and the parallel update
    double uparb = 0.0;
    {
        Point<D, kYee> p;
        Smp s;
        LocalD L;
        sample_at(acc, pc, st, p);
        to_sample(p, s);
        local_fields(s.E, s.B, K, L);
        if (curv) curvature_scalars_dir(s, K, L);
        LocalBar Lb;
        SampleBar<D> sb;
        double Ab, Cb;
        drift_back<D>(s, L, pc, upn, mu, inv_qm, curv, K, Fnb, Lb, sb, upnb, mub);
        parallel_back(L, upar, mu, qm, curv, K, upnb, Lb, uparb, mub, Ab, Cb);
        if (curv) scalars_back<D>(s, L, pc, K, Ab, Cb, Lb, sb);
        local_back<D>(s, L, K, Lb, sb);
        point_back<D, kYee>(win, pc, st, p, sb, xb);
    }

    // 1. decomposition at R^{n-1/2}
    {
        Point<D, kYee> p;
        Smp s;
        LocalD L;
        sample_at(acc, pc, Rh, p);
        to_sample(p, s);
        local_fields(s.E, s.B, K, L);
        LocalBar Lb;
        SampleBar<D> sb;
        const Gam<double> G = gamma_full2(u[0], u[1], u[2], K);
        double vc[3] = {0.0, 0.0, 0.0}, up[3];
        if (curv) v_curv_dir(L, s, upar, G.inv, inv_qm, K, vc);
#pragma unroll
        for (int i = 0; i < 3; ++i) up[i] = (u[i] - upar * L.b[i]) - (L.vE[i] + vc[i]) * G.g;
        const double up2 = dot3(up, up);
        const double inv_nu = up2 > 0.0 ? rsqrt_nr(up2) : 0.0;
        const double d = dot3(bp, bpb);
        const double muk = mub * L.inv_kappa;
        const double up2b = muk * (0.5 * L.inv_B);
        Lb.inv_B += muk * (0.5 * up2);
        Lb.kappa -= muk * mu;
        double gfb = 0.0, igb = 0.0, vcb[3], uvb[3], upb[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            upb[i] = (bpb[i] - bp[i] * d) * inv_nu + (2.0 * up2b) * up[i];
            uparb -= L.b[i] * upb[i];
            Lb.b[i] -= upar * upb[i];
            vcb[i] = -G.g * upb[i];
            Lb.vE[i] += vcb[i];
            gfb -= (L.vE[i] + vc[i]) * upb[i];
        }
        if (curv) vcurv_back<D>(s, L, pc, upar, G.inv, inv_qm, K, vcb, Lb, sb, uparb, igb);
        gfb -= igb * (G.inv * G.inv);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            uvb[i] = (upb[i] + (gfb * K.inv_c2 * G.inv) * u[i]) + uparb * L.b[i];
            Lb.b[i] += uparb * u[i];
        }
        local_back<D>(s, L, K, Lb, sb);
        double Rhb[D];
#pragma unroll
        for (int a = 0; a < D; ++a) Rhb[a] = 0.0;
        point_back<D, kYee>(win, pc, Rh, p, sb, Rhb);
#pragma unroll
        for (int a = 0; a < D; ++a) {
            lam[a] = xb[a] + 0.5 * Rhb[a];
            lam[D + a] = 0.5 * Rhb[a];
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) lam[2 * D + i] = uvb[i];
    }
}

}  // namespace adj
}  // namespace gcb
