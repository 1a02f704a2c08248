"""The production arithmetic at the ends of binary64's range, against the parity
arithmetic on the same inputs: momenta whose square overflows (Gamma infinite, no
rotation, the electric kick alone), and switch limits f_E whose square leaves the
range (E/B < f_E decides, as stated, not the squares)."""
import numpy as np
import pytest
import torch

from gpu_util import GpuRun
from test_gpu_3d import GpuRun3
from test_gpu_gr import GrRun, to_device
from workloads import make_config, make_config3, make_gr_config

pytestmark = pytest.mark.gpu

E0, B0 = (0.01, -0.02, 0.03), (0.3, 0.2, 0.5)


def uniform(dim, E=E0, B=B0):
    """A run with uniform fields."""
    cfg = make_config("harris64") if dim == 2 else make_config3("harris3d32")
    F = np.ones_like(cfg.fields()) * np.array(E + B).reshape((6,) + (1,) * dim)
    return cfg, (GpuRun if dim == 2 else GpuRun3)(cfg, F)


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("kernel,sort,tile", [(1, 0, 0), (2, 1, 4)])
def test_overflowing_momentum(dim, kernel, sort, tile):
    from paper_2007_14401_amd import gcb, state
    cfg, run = uniform(dim)
    try:
        out = {}
        for arith in (gcb.GCB_ARITH_EXACT, gcb.GCB_ARITH_FAST):
            ens = cfg.particles(n=130)
            ens.ux[:] = np.where(np.arange(130) % 3 == 0, 1e160, 1e153)
            ens.uy[::2] = -1e155
            t = state.to_device(ens)
            run.push(t, 1, kernel=kernel, sort_every=sort, tile=tile, arith=arith)
            out[arith] = state.unsort(t)
    finally:
        run.close()
    for k in ("ux", "uy", "uz"):
        a, b = out[gcb.GCB_ARITH_EXACT][k], out[gcb.GCB_ARITH_FAST][k]
        assert np.isfinite(b).all(), k
        # a handful of roundings of terms of order one, or of the component itself
        assert np.allclose(b, a, rtol=1e-14, atol=1e-14), k


# scales of E and B, f_E, f_rho, and whether the guiding-center branch may be taken
SWITCH = {"no E": (0.0, 1.0, 1e-170, 0.4, True), "E/B below": (1e-20, 1e150, 1e-165, 0.4, True),
          "E/B above": (1e-20, 1e150, 1e-175, 0.4, False),
          "large f_E": (1.0, 1e-160, 1e200, np.inf, True), "f_E 0": (0.0, 1.0, 0.0, 0.4, False)}


@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("case", SWITCH)
def test_extreme_switch_limit(dim, case):
    from paper_2007_14401_amd import gcb, state
    e, b, f_E, f_rho, gca = SWITCH[case]
    cfg, run = uniform(dim, tuple(e * np.array(E0)), tuple(b * np.array(B0)))
    try:
        tr = {}
        for arith in (gcb.GCB_ARITH_EXACT, gcb.GCB_ARITH_FAST):
            t = state.to_device(cfg.particles(n=130))
            tr[arith] = run.push(t, 1, trace=True, f_E=f_E, f_rho=f_rho,
                                 arith=arith)[0].cpu().numpy()
    finally:
        run.close()
    assert (tr[gcb.GCB_ARITH_EXACT] == 0).any() == gca
    assert np.array_equal(tr[gcb.GCB_ARITH_EXACT], tr[gcb.GCB_ARITH_FAST])


def test_extreme_switch_limit_curved():
    from paper_2007_14401_amd import gcb
    cfg = make_gr_config("grbh64")
    F = cfg.fields()
    F[:3] = 0.0
    run = GrRun(cfg, F)
    try:
        tr = [run.push(to_device(cfg.particles(n=130)), 1, f_E=1e-170, arith=a)[0].cpu().numpy()
              for a in (gcb.GCB_ARITH_EXACT, gcb.GCB_ARITH_FAST)]
    finally:
        run.close()
    assert (tr[0] == 0).any()
    assert np.array_equal(tr[0], tr[1])


@pytest.mark.parametrize("dim", [2, 3])
def test_overflowing_momentum_backwards(dim):
    """One step backwards in uniform fields: a particle whose u^2 overflows does not
    move or turn, so its cotangents pass through, and no node of the field cotangents
    is lost to it."""
    from paper_2007_14401_amd import gcb, state
    cfg, run = uniform(dim)
    n, k = 130, 2 * dim + 3
    rng = np.random.default_rng(2)
    lam = rng.normal(size=(k, n))
    dev = lambda a, t=torch.float64: torch.as_tensor(a, dtype=t, device="cuda:0")
    try:
        ens = cfg.particles(n=n)
        ens.ux[::3] = 1e160
        t = state.to_device(ens)
        end, start = [dev(v) for v in lam], [dev(0 * v) for v in lam]
        F = run.cfg.fields()[0]
        d = [dev(0 * F, torch.float32) for _ in range(6)]
        parts = gcb.particles(t) if dim == 2 else gcb.particles3(t)
        back = gcb.gcb_push_backward if dim == 2 else gcb.gcb_push_backward_3d
        prm = gcb.params(dt=cfg.dt, c=cfg.c, qm=cfg.qm, f_rho=cfg.f_rho, f_E=cfg.f_E)
        back(run.ctx, parts, prm, 1, end, start, d[:3], d[3:])
        torch.cuda.synchronize()
        got = np.stack([v.cpu().numpy() for v in start])
        nodes = np.stack([v.cpu().numpy() for v in d])
    finally:
        run.close()
    assert np.isfinite(got).all() and np.isfinite(nodes).all()
    want = lam[:, ::3].copy()
    want[:dim] += want[dim:2 * dim]
    want[dim:2 * dim] = 0.0
    assert np.array_equal(got[:, ::3], want)
