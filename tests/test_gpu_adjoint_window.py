"""Batches, chunks and the LDS window of the reverse sweep against the oracle
gradient, where they can go wrong: more particles in a tile than a chunk takes
(64 of these small ensembles), more steps than a batch, a grid smaller than the
window, drifts that leave the window within one step, the collocated lattice,
and the smallest and largest number of iterations.

Tolerances as for the other adjoint tests: 1e-8 of the largest entry per state
cotangent (binary64 recurrences in another order), 2e-5 for the field
cotangents (binary32 grid).  None of these runs amplifies a change of 1e-13 in
the start positions to more than 1e-10 of a cotangent."""
import numpy as np
import pytest

import oracle as O
from gpu_util import log, oracle_params
from workloads import make_config, make_config3

pytestmark = pytest.mark.gpu

COLLOCATED = tuple((0.0, 0.0) for _ in range(6))
COLLOCATED3 = tuple((0.0, 0.0, 0.0) for _ in range(6))

CASES2 = {
    "batches": (dict(), 333, 27),
    "small grid": (dict(nx=20, ny=40), 150, 14),
    "leaves the window": (dict(dt=7.0), 200, 3),
    "collocated": (dict(stagger=COLLOCATED), 200, 6),
    "collocated, small grid, leaves the window": (
        dict(stagger=COLLOCATED, nx=20, ny=40, dt=7.0), 100, 3),
    "one iteration": (dict(n_iter=1), 130, 6),
    "eight iterations": (dict(n_iter=8), 65, 6),
    "one particle": (dict(), 1, 13),
}
CASES3 = {
    "batches": (dict(), 150, 9),
    "small grid": (dict(nx=9, nz=8), 300, 6),
    "leaves the window": (dict(dt=4.0), 150, 3),
    "collocated": (dict(stagger=COLLOCATED3), 100, 3),
    "eight iterations": (dict(n_iter=8), 65, 3),
}


def reference(dim, case):
    over, n, steps = (CASES2 if dim == 2 else CASES3)[case]
    cfg = make_config("harris64", **over) if dim == 2 else make_config3("harris3d32", **over)
    return cfg, cfg.fields(), cfg.particles(n=n, seed_offset=41), steps


def oracle_gradient(dim, cfg, F, ens, steps):
    if dim == 2:
        return O.push_gradients(F, cfg.dx, cfg.dy, cfg.stagger, O.State.from_numpy(ens),
                                oracle_params(cfg), steps)
    p = O.Params3(dt=cfg.dt, c=cfg.c, f_rho=cfg.f_rho, f_E=cfg.f_E,
                  curvature=bool(cfg.curvature), n_iter=cfg.n_iter, Lx=cfg.Lx, Ly=cfg.Ly,
                  Lz=cfg.Lz, dl=cfg.dl)
    return O.push_gradients3(F, cfg.dx, cfg.dy, cfg.dz, cfg.stagger, O.State3.from_numpy(ens),
                             p, steps)


@pytest.mark.parametrize("dim,case", [(2, c) for c in CASES2] + [(3, c) for c in CASES3])
def test_reverse_sweep_matches_oracle(dim, case, monkeypatch):
    from paper_2007_14401_amd import autograd as A
    from test_gpu_adjoint import NAMES, _grad_gpu
    from test_gpu_adjoint3 import NAMES3, _grad_gpu3
    cfg, F, ens, steps = reference(dim, case)
    # the 2D helper's context loads the Yee lattice unless told otherwise
    load = A.PushContext.load
    monkeypatch.setattr(A.PushContext, "load",
                        lambda self, E, B: load(self, E, B, stagger=cfg.stagger))
    log(f"{dim}d {case}: gpu")
    _, g, gF = (_grad_gpu if dim == 2 else _grad_gpu3)(cfg, F, ens, steps, steps)
    log(f"{dim}d {case}: oracle")
    ref = oracle_gradient(dim, cfg, F, ens, steps)
    for k in NAMES if dim == 2 else NAMES3:
        a, b = g[k], ref["d" + k].numpy()
        err = np.max(np.abs(a - b)) / np.max(np.abs(b))
        assert err <= 1e-8, (k, err)
    b = ref["dF"].numpy()
    err = np.max(np.abs(gF - b)) / np.max(np.abs(b))
    log(f"{dim}d {case} dF: max-norm rel err {err:.2e}")
    assert err <= 2e-5
