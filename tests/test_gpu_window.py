"""The LDS window of the tiled pushes: at the edges of tiles and of the window,
across the periodic edge, for windows as large as the box, the tiled kernel
(in place) gives what the cache-served kernel gives, bit for bit in the parity
arithmetic; the status bytes differ in the window-miss bit alone."""
import numpy as np
import pytest
import torch

from tests.gpu_util import log
from workloads import make_config
from workloads.configs3d import make_config3

pytestmark = pytest.mark.gpu


def _edges(n, tile, rng, count):
    """Coordinates on tile edges, half cells, next to them and next to the box
    edge, shuffled."""
    e = np.arange(0, n, tile, dtype=np.float64)
    base = np.concatenate([e, e + 0.5, [0.0, n - 0.5]])
    x = np.concatenate([base, np.nextafter(base, -1.0), np.nextafter(base, n), base + 0.25])
    x = np.concatenate([x, rng.uniform(0.0, n, count)])
    return np.mod(rng.choice(x, count), n)


def _push(gcb, call, ctx, parts_of, t, prm, steps):
    call(ctx, parts_of(t), prm, steps)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in t.items() if v is not None}


def _same(a, b):
    for k in a:
        if k == "status":
            assert np.array_equal(a[k] & ~np.uint8(32), b[k] & ~np.uint8(32))
        else:
            assert np.array_equal(a[k], b[k], equal_nan=True), k


@pytest.mark.parametrize("nx,ny,tile,sort,steps", [
    (64, 48, 16, 4, 8), (50, 37, 24, 4, 4), (33, 35, 2, 1, 3), (64, 64, 40, 4, 4),
    (20, 21, 20, 10, 10)])
@pytest.mark.parametrize("stagger", ["yee", "collocated"])
def test_window_2d(nx, ny, tile, sort, steps, stagger):
    from paper_2007_14401_amd import gcb, state
    cfg = make_config("harris64", nx=nx, ny=ny, n=3001,
                      stagger=gcb.YEE_STAGGER if stagger == "yee" else ((0.0, 0.0),) * 6)
    rng = np.random.default_rng(7)
    F, ens = cfg.fields(), cfg.particles()
    ens.x, ens.y = _edges(nx, tile, rng, cfg.n), _edges(ny, tile, rng, cfg.n)
    ens.xp, ens.yp = np.mod(ens.x - 0.3, nx), np.mod(ens.y + 0.2, ny)
    ctx = gcb.gcb_create(0)
    gcb.gcb_load_fields(ctx, gcb.grid_desc(nx, ny, stagger=cfg.stagger), [F[0], F[1], F[2]],
                        [F[3], F[4], F[5]])
    kw = dict(dt=cfg.dt, c=cfg.c, qm=cfg.qm, f_rho=cfg.f_rho, f_E=cfg.f_E)
    try:
        tiled = gcb.params(sort_every=sort, tile=tile, kernel=gcb.GCB_KERNEL_AUTO, keep_order=1,
                           **kw)
        plain = gcb.params(kernel=gcb.GCB_KERNEL_GLOBAL, **kw)
        a = _push(gcb, gcb.gcb_push, ctx, gcb.particles, state.to_device(ens), tiled, steps)
        b = _push(gcb, gcb.gcb_push, ctx, gcb.particles, state.to_device(ens), plain, steps)
    finally:
        gcb.gcb_destroy(ctx)
    log(f"window {nx}x{ny} tile {tile}: {int((a['status'] & 32 > 0).sum())} misses")
    _same(a, b)


@pytest.mark.parametrize("n3,tile,sort,steps", [
    ((20, 24, 18), 4, 4, 8), ((13, 9, 11), 6, 2, 4), ((9, 10, 8), 2, 1, 2)])
def test_window_3d(n3, tile, sort, steps):
    from paper_2007_14401_amd import gcb, state
    cfg = make_config3("harris3d32", nx=n3[0], ny=n3[1], nz=n3[2], n=2001)
    rng = np.random.default_rng(8)
    F, ens = cfg.fields(), cfg.particles()
    ens.x, ens.y, ens.z = (_edges(m, tile, rng, cfg.n) for m in n3)
    ens.xp, ens.yp, ens.zp = (np.mod(v - 0.2, m) for v, m in zip((ens.x, ens.y, ens.z), n3))
    ctx = gcb.gcb_create(0)
    gcb.gcb_load_fields_3d(ctx, gcb.grid3_desc(*n3), [F[0], F[1], F[2]], [F[3], F[4], F[5]])
    kw = dict(dt=cfg.dt, c=cfg.c, qm=cfg.qm, f_rho=cfg.f_rho, f_E=cfg.f_E)
    try:
        tiled = gcb.params(sort_every=sort, tile=tile, keep_order=1, **kw)
        plain = gcb.params(kernel=gcb.GCB_KERNEL_GLOBAL, **kw)
        a = _push(gcb, gcb.gcb_push_3d, ctx, gcb.particles3, state.to_device(ens), tiled, steps)
        b = _push(gcb, gcb.gcb_push_3d, ctx, gcb.particles3, state.to_device(ens), plain, steps)
    finally:
        gcb.gcb_destroy(ctx)
    _same(a, b)
