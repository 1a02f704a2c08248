"""The production arithmetic at the ends of binary64's range, against the parity
arithmetic on the same inputs: momenta whose square overflows (Gamma infinite, no
rotation, the electric kick alone)."""
import numpy as np
import pytest
import torch

from gpu_util import GpuRun
from test_gpu_3d import GpuRun3
from workloads import make_config, make_config3

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
