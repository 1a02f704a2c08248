"""The LDS window of the tiled kernel itself (GCB_KERNEL_TILED: a window that does
not fit is an error, not the other kernel), in place, over particles at the edges of
tiles, of cells and of the box, and with midpoints far enough behind the
particle to leave the window, which has to be seen in the status bytes.

Parity arithmetic: what the cache-served kernel gives, bit for bit, over several
steps.  Production arithmetic, which reads the window's layout its own way: one
step within its stated 1e-12 of the parity arithmetic's, with the same switch
decisions."""
import numpy as np
import pytest
import torch

from gpu_util import log
from test_gpu_window import _edges
from workloads import make_config, make_config3

pytestmark = pytest.mark.gpu

HALO = 32
# box, tile, sort interval, steps; cells that the previous position lies behind
CASES2 = [((64, 48), 16, 4, 8, 0.3), ((50, 37), 24, 4, 4, 0.3), ((33, 35), 2, 1, 3, 0.3),
          ((64, 64), 40, 4, 4, 9.0), ((65, 90), 16, 2, 2, 14.0), ((20, 21), 20, 10, 10, 0.3)]
CASES3 = [((20, 24, 18), 4, 4, 8, 0.2), ((13, 9, 11), 6, 2, 4, 0.2), ((9, 10, 8), 2, 1, 2, 0.2),
          ((30, 29, 28), 4, 2, 2, 10.0)]


def setup(dim, size, tile, behind, stagger="yee"):
    from paper_2007_14401_amd import gcb
    yee = gcb.YEE_STAGGER if dim == 2 else gcb.YEE3_STAGGER
    lattice = yee if stagger == "yee" else ((0.0,) * dim,) * 6
    over = dict(zip(("nx", "ny", "nz"), size), n=3001, stagger=lattice)
    cfg = make_config("harris64", **over) if dim == 2 else make_config3("harris3d32", **over)
    rng = np.random.default_rng(7)
    F, ens = cfg.fields(), cfg.particles()
    for a, m in zip("xyz", size):
        v = _edges(m, tile, rng, cfg.n)
        setattr(ens, a, v)
        setattr(ens, a + "p", np.mod(v - behind, m))
    ctx = gcb.gcb_create(0)
    E, B = [F[0], F[1], F[2]], [F[3], F[4], F[5]]
    if dim == 2:
        gcb.gcb_load_fields(ctx, gcb.grid_desc(*size, stagger=lattice), E, B)
    else:
        gcb.gcb_load_fields_3d(ctx, gcb.grid3_desc(*size, stagger=lattice), E, B)
    kw = dict(dt=cfg.dt, c=cfg.c, qm=cfg.qm, f_rho=cfg.f_rho, f_E=cfg.f_E)
    return cfg, ctx, ens, kw


def push(dim, ctx, ens, steps, **kw):
    from paper_2007_14401_amd import gcb, state
    t = state.to_device(ens)
    trace = torch.zeros((steps, t["x"].shape[0]), dtype=torch.uint8, device="cuda")
    parts = gcb.particles(t) if dim == 2 else gcb.particles3(t)
    (gcb.gcb_push if dim == 2 else gcb.gcb_push_3d)(ctx, parts, gcb.params(**kw), steps,
                                                    s_trace=trace)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in t.items() if v is not None}, trace.cpu().numpy()


@pytest.mark.parametrize("stagger", ["yee", "collocated"])
@pytest.mark.parametrize("dim,case", [(2, c) for c in CASES2] + [(3, c) for c in CASES3])
def test_tiled_window(dim, case, stagger):
    from paper_2007_14401_amd import gcb
    size, tile, sort, steps, behind = case
    cfg, ctx, ens, kw = setup(dim, size, tile, behind, stagger)
    tiled = dict(kernel=gcb.GCB_KERNEL_TILED, sort_every=sort, tile=tile, keep_order=1, **kw)
    plain = dict(kernel=gcb.GCB_KERNEL_GLOBAL, **kw)
    try:
        a, ta = push(dim, ctx, ens, steps, **tiled)
        b, tb = push(dim, ctx, ens, steps, **plain)
        b1, tb1 = push(dim, ctx, ens, 1, **plain)
        f, tf = push(dim, ctx, ens, 1, arith=gcb.GCB_ARITH_FAST, **tiled)
    finally:
        gcb.gcb_destroy(ctx)
    misses = int((a["status"] & HALO > 0).sum())
    log(f"{dim}d {size} tile {tile} behind {behind}: {misses} misses")
    if behind > 1.0:
        assert misses > 0 and (f["status"] & HALO > 0).any()
    for k in a:
        if k != "status":
            assert np.array_equal(a[k], b[k], equal_nan=True), k
    assert np.array_equal(a["status"] & ~np.uint8(HALO), b["status"])
    assert np.array_equal(ta, tb)

    assert np.array_equal(tf, tb1)
    for k in ("x", "y", "z", "xp", "yp", "zp", "ux", "uy", "uz"):
        if k not in f:
            continue
        d, floor = np.abs(f[k] - b1[k]), cfg.c if k[0] == "u" else 1.0
        if k[0] != "u":
            L = size["xyz".index(k[0])]
            d = np.minimum(d, L - d)
        assert np.max(d / np.maximum(np.abs(b1[k]), floor)) <= 1e-12, k
