"""The reverse sweep over a box with few particles per tile, which has them gather
from and add to the grid instead of a window: against the oracle gradient (Yee
and collocated lattices, points across the periodic edges), and, where crowded
tiles keep their windows beside it, bit for bit what the windows give the same
particles in a call of fewer.

Tolerances as for the other adjoint tests: 1e-8 of the largest entry per state
cotangent, 2e-5 for the field cotangents (binary32 outputs)."""
import numpy as np
import pytest
import torch

import oracle as O
from gpu_util import log, oracle_params
from test_gpu_adjoint_window import COLLOCATED, COLLOCATED3, oracle_gradient
from workloads import make_config, make_config3

pytestmark = pytest.mark.gpu

# more than 2048 tiles (32 cells in 2D, 6 in 3D) and particles
SIZES = {2: (1470, 1530), 3: (80, 85, 90)}


def config(dim, **over):
    if dim == 2:
        return make_config("harris64", nx=SIZES[2][0], ny=SIZES[2][1], **over)
    nx, ny, nz = SIZES[3]
    return make_config3("harris3d32", nx=nx, ny=ny, nz=nz, **over)


@pytest.mark.parametrize("dim,lattice", [(2, "yee"), (2, "collocated"), (3, "yee"),
                                         (3, "collocated")])
def test_sparse_box_matches_oracle(dim, lattice, monkeypatch):
    from paper_2007_14401_amd import autograd as A
    from test_gpu_adjoint import NAMES, _grad_gpu
    from test_gpu_adjoint3 import NAMES3, _grad_gpu3
    over = {} if lattice == "yee" else dict(stagger=COLLOCATED if dim == 2 else COLLOCATED3)
    cfg = config(dim, **over)
    load = A.PushContext.load
    monkeypatch.setattr(A.PushContext, "load",
                        lambda self, E, B: load(self, E, B, stagger=cfg.stagger))
    F, steps = cfg.fields(), 2
    ens = cfg.particles(n=2100, seed_offset=43)
    ens.x[:40] = np.mod(ens.x[:40] / cfg.Lx - 0.5, cfg.Lx)   # about the edges
    ens.y[20:60] = np.mod(ens.y[20:60] / cfg.Ly - 0.5, cfg.Ly)
    ens.xp[:60], ens.yp[:60] = ens.x[:60], ens.y[:60]
    log(f"{dim}d {lattice}: gpu")
    _, g, gF = (_grad_gpu if dim == 2 else _grad_gpu3)(cfg, F, ens, steps, steps)
    log(f"{dim}d {lattice}: oracle")
    ref = oracle_gradient(dim, cfg, F, ens, steps)
    for k in NAMES if dim == 2 else NAMES3:
        a, b = g[k], ref["d" + k].numpy()
        err = np.max(np.abs(a - b)) / np.max(np.abs(b))
        assert err <= 1e-8, (k, err)
    b = ref["dF"].numpy()
    err = np.max(np.abs(gF - b)) / np.max(np.abs(b))
    log(f"{dim}d {lattice} dF: max-norm rel err {err:.2e}")
    assert err <= 2e-5


@pytest.mark.parametrize("dim,size", [(2, (2080, 2080)), (3, (80, 85, 90))])
@pytest.mark.parametrize("crowd", [0, 64, 500])
def test_windows_and_grid_give_the_same_bits(dim, size, crowd):
    """2000 particles alone (at most 2048: a window each), and with others beside
    them: `crowd` in each of three tiles and some in the box."""
    from paper_2007_14401_amd import gcb
    rng = np.random.default_rng(9)
    few, more, k, steps, tile = 2000, 400, 2 * dim + 3, 5, 32 if dim == 2 else 6
    n = few + more + 3 * crowd
    pos = np.stack([rng.uniform(0, m, n) for m in size])
    for c in range(3):
        at = few + more + c * crowd
        for a in range(dim):
            pos[a, at:at + crowd] = (c + 1) * tile + tile * rng.uniform(0, 1, crowd)
    u = rng.normal(0, 0.3, (3, n))
    prev = np.mod(pos - 0.3 * rng.normal(0, 1, (dim, n)), np.array(size)[:, None])
    F = rng.normal(0, 0.1, (6,) + size[::-1])
    F[3:] += np.array([0.3, 0.2, 1.0]).reshape((3,) + (1,) * dim)
    lam = rng.normal(size=(k, n))
    dev = lambda a, t=torch.float64: torch.as_tensor(np.ascontiguousarray(a), dtype=t,
                                                     device="cuda:0")
    ctx = gcb.gcb_create(0)
    try:
        Fd = dev(F)
        E, B = [Fd[i] for i in range(3)], [Fd[i] for i in range(3, 6)]
        if dim == 2:
            gcb.gcb_load_fields(ctx, gcb.grid_desc(*size), E, B)
        else:
            gcb.gcb_load_fields_3d(ctx, gcb.grid3_desc(*size), E, B)
        prm = gcb.params(qm=-1.0, sort_every=4, tile=20 if dim == 2 else 4)
        out = {}
        for m in (few, n):
            names = ["x", "y", "z"][:dim]
            t = {a: dev(pos[i, :m]) for i, a in enumerate(names)}
            t.update({a + "p": dev(prev[i, :m]) for i, a in enumerate(names)})
            t.update({a: dev(u[i, :m]) for i, a in enumerate(("ux", "uy", "uz"))})
            t["status"] = torch.zeros(m, dtype=torch.uint8, device="cuda:0")
            end, start = [dev(v[:m]) for v in lam], [dev(0 * v[:m]) for v in lam]
            d = [torch.zeros(F[0].size, dtype=torch.float32, device="cuda:0") for _ in range(6)]
            log(f"{dim}d crowd {crowd}: {m} particles")
            parts = gcb.particles(t) if dim == 2 else gcb.particles3(t)
            back = gcb.gcb_push_backward if dim == 2 else gcb.gcb_push_backward_3d
            back(ctx, parts, prm, steps, end, start, d[:3], d[3:])
            torch.cuda.synchronize()
            out[m] = np.stack([v.cpu().numpy() for v in start])
            nodes = torch.stack(d).abs().sum(1)
            assert torch.isfinite(nodes).all() and (nodes > 0).all()
    finally:
        gcb.gcb_destroy(ctx)
    assert np.isfinite(out[few]).all() and np.abs(out[few]).max() > 0
    assert np.array_equal(out[few], out[n][:, :few])
