"""The reverse sweep's particle cotangents against the same step in 80 bits, on
the host.  The sweep is the same for every caller, so its arithmetic (contracted
multiply-adds, refined reciprocals) may be no less exact than correctly rounded
operations without contraction: the root mean square over the particles of the
error of the u cotangents and of all seven, relative to the norm of each
particle's, is held to what that evaluation of the same derivative has on these
inputs."""
import ctypes

import numpy as np
import pytest

from host_arith import compile_host
from workloads import make_config

SOURCE = """
#define GCB_ARITH_NS arith_fast
#define GCB_FAST_ARITH 1
#include <hip/hip_runtime.h>
#include <cmath>
#include <vector>
typedef double in64;
#ifdef EXTENDED
using std::fabs; using std::floor; using std::sqrt; using std::fma; using std::fmin; using std::fmax;
#define double long double
#endif
#include "gcb_adjoint.hpp"
using namespace gcb;
struct NoNodes {   // the node cotangents are not looked at here
    template <bool kYee>
    void add(const PushConst&, const double*, const adj::Point<2, kYee>&,
             const adj::SampleBar<2>&) const {}
};
// one step of n particles: st, lam (7 values each); S 1 = Boris, written when `decide`
extern "C" void step(const in64* F_, int nx, int ny, const in64* par, const in64* st_,
                     const in64* qm, unsigned char* S, long n, in64* lam, in64* rest,
                     int decide) {
    PushConst pc{};
    pc.dt = par[0]; pc.c = par[1]; pc.f_rho = par[2]; pc.f_E = par[3];
    pc.curvature = (int)par[4]; pc.n_iter = (int)par[5];
    pc.c2 = pc.c2_inv_dl = pc.c * pc.c; pc.inv_c2 = 1 / (pc.c * pc.c);
    pc.inv_dx = pc.inv_dy = pc.inv_dl = 1; pc.nx = nx; pc.ny = ny; pc.Lx = nx; pc.Ly = ny;
    pc.inv_Lx = 1 / pc.Lx; pc.inv_Ly = 1 / pc.Ly;
    const int W = 40, o[2] = {-4, -4};
    std::vector<double> F(F_, F_ + (size_t)6 * nx * ny), lds((size_t)6 * W * W);
    for (int j = 0; j < W; ++j) for (int i = 0; i < W; ++i) for (int k = 0; k < 6; ++k)
        lds[window_elem<double>(k, j * W + i, W * W)] =
            F[((size_t)wrap_index(j - 4, ny) * nx + wrap_index(i - 4, nx)) * 6 + k];
    const auto acc = adj::Dim<2>::acc(lds.data(), F.data(), pc, o, W);
    const auto K = adj::Dim<2>::consts(pc);
    for (long p = 0; p < n; ++p) {
        double st[7], l[7];
        for (int c = 0; c < 7; ++c) { st[c] = st_[p * 7 + c]; l[c] = lam[p * 7 + c]; }
        if (decide) {
            Sample<double> s;
            gather<double, true, true>(acc, pc, K, st[0], st[1], s);
            S[p] = switch_gca_f64(s.E, s.B, st[4], st[5], st[6], (double)qm[p], pc) ? 0 : 1;
        }
        if (S[p] == 0) adj::gca_vjp<2, true>(acc, NoNodes(), pc, K, st, (double)qm[p], l);
        else adj::boris_vjp<2, true>(acc, NoNodes(), pc, K, st, (double)qm[p], l);
        for (int c = 0; c < 7; ++c) {
            lam[p * 7 + c] = (in64)l[c];
            rest[p * 7 + c] = (in64)(l[c] - (double)(in64)l[c]);
        }
    }
}
"""


@pytest.fixture(scope="module")
def libs(tmp_path_factory):
    return (compile_host(str(tmp_path_factory.mktemp("v64")), SOURCE, "-ffp-contract=on"),
            compile_host(str(tmp_path_factory.mktemp("v80")), SOURCE, "-ffp-contract=off",
                         "-DEXTENDED"))


def _step(lib, F, cfg, st, qm, S, lam, decide):
    par = np.array([cfg.dt, cfg.c, cfg.f_rho, cfg.f_E, cfg.curvature, cfg.n_iter], float)
    lam, rest = lam.copy(), np.zeros_like(lam)
    p = [a.ctypes.data_as(ctypes.c_void_p) for a in (F, par, st, qm, S, lam, rest)]
    lib.step(p[0], cfg.nx, cfg.ny, p[1], p[2], p[3], p[4], ctypes.c_long(len(st)), p[5], p[6],
             int(decide))
    return lam, rest


# root mean square errors of the correctly rounded evaluation: u, all
IEEE = {"boris": (1.53e-16, 1.27e-16), "guiding center": (2.99e-16, 2.30e-16)}


def test_cotangents_no_less_exact_than_rounded_operations(libs):
    cfg = make_config("harris64")
    F = np.ascontiguousarray(np.moveaxis(cfg.fields(), 0, -1))
    e = cfg.particles(n=20000)
    st = np.ascontiguousarray(np.stack([e.x, e.y, e.xp, e.yp, e.ux, e.uy, e.uz], 1))
    qm = np.full(20000, float(cfg.qm))
    lam = np.random.default_rng(3).normal(size=(20000, 7))
    S = np.zeros(20000, np.uint8)
    got, _ = _step(libs[0], F, cfg, st, qm, S, lam, True)
    ref, rest = _step(libs[1], F, cfg, st, qm, S, lam, False)
    err = (got - ref) - rest
    for s, name in ((1, "boris"), (0, "guiding center")):
        m = S == s
        assert m.sum() > 5000
        for sl, what, bound in ((slice(4, 7), "u", IEEE[name][0]),
                                (slice(0, 7), "all", IEEE[name][1])):
            r = np.linalg.norm(err[m, sl], axis=1) / np.linalg.norm(ref[m, sl], axis=1)
            rms = float(np.sqrt(np.mean(r * r)))
            print(f"{name}, {what}: rms {rms:.3e} (bound {bound:.3e})")
            assert rms <= bound, (name, what)
