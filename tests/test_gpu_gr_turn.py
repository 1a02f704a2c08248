"""The production curved-spacetime step takes the midpoints' sine and cosine of
theta from the step start's while they lie within 1/16, and evaluates them
otherwise.  One step at time steps where all, or most, midpoints do, with two
to six iterations, against the oracle: per particle within
max(1e-12, 10 x the oracle's own deviation when its start is moved by up to
four units in the last place), as in the production form's other tests, and
the oracle's switch decisions."""
import numpy as np
import pytest

from oracle import gr
from test_gpu_gr import NAMES, GrRun, run_oracle, to_device
from test_gpu_gr_production import FAST, _nudge, chaos_aware_check
from workloads import make_gr_config

pytestmark = pytest.mark.gpu

CASES = [(0.02, 4), (2.0, 4), (8.0, 2), (8.0, 6)]


def start(dt, n_iter):
    cfg = make_gr_config("grbh64", dt=dt, n_iter=n_iter)
    return cfg, cfg.fields(), cfg.particles(n=2000, seed_offset=51)


def nudged(cfg, F, e):
    metric = gr.KerrSchild(cfg.a)
    grid = gr.GRGrid(F, cfg.r_min, cfg.r_max)
    dl = gr.cell_lengths(metric, grid)
    p = gr.GRParams(dt=cfg.dt, f_rho=cfg.f_rho, f_E=cfg.f_E, n_iter=cfg.n_iter)
    out = []
    for seed in (1, 2, 3):
        rng = np.random.default_rng(seed)
        st = gr.GRState.from_numpy(e)
        for k in NAMES:
            setattr(st, k, _nudge(getattr(st, k), rng))
        out.append(gr.step(metric, grid, dl, st, p)[0])
    return out


@pytest.mark.parametrize("dt,n_iter", CASES)
def test_midpoint_angles(dt, n_iter):
    cfg, F, e = start(dt, n_iter)
    run = GrRun(cfg, F)
    try:
        t = to_device(e)
        tr, _ = run.push(t, 1, arith=FAST)
        got = {k: t[k].cpu().numpy() for k in NAMES}
        tr = np.asarray(tr.cpu() if hasattr(tr, "cpu") else tr)
    finally:
        run.close()
    ref, S, _ = run_oracle(cfg, F, e, 1)
    chaos_aware_check(got, tr.reshape(1, -1), ref, S.reshape(1, -1), nudged(cfg, F, e),
                      f"dt {dt}, K {n_iter}")
