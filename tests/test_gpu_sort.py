"""The cell sort at the edges of its paths: one bucket level (up to 256 tiles),
two (up to 65536) and the radix passes beyond; the particle counts where the
block size and the scan change; every particle in one tile.  Index work: the
order is the stable order by tile, exactly, and every array of the state has
moved along (and is back in the caller's buffers after an odd number of
sorts)."""
import numpy as np
import pytest
import torch

from gpu_util import GpuRun, log
from workloads import make_config

pytestmark = pytest.mark.gpu

# (nx, ny, tile): 16, 256, 272, 3072 and 69632 tiles
GRIDS = [(64, 64, 16), (128, 128, 8), (136, 128, 8), (512, 384, 8), (1088, 1024, 4)]
COUNTS = [1, 1000, 4097, 262144, 262145, 1048577]


@pytest.mark.parametrize("nx,ny,tile", GRIDS)
def test_cell_sort_paths(nx, ny, tile):
    cfg = make_config("harris64", nx=nx, ny=ny)
    run = GpuRun(cfg, cfg.fields())
    rng = np.random.default_rng(nx + tile)
    try:
        for n, spread in [(c, "all") for c in COUNTS] + [(50000, "one tile"), (50000, "few")]:
            log(f"{nx}x{ny} tile {tile}: {n} {spread}")
            x = rng.uniform(0, cfg.Lx, n)
            y = rng.uniform(0, cfg.Ly, n)
            if spread == "one tile":
                x, y = 2 * tile + x % tile, tile + y % tile
            elif spread == "few":
                x, y = x % (2 * tile), cfg.Ly - 1 - y % (2 * tile)
            u = rng.normal(0, 1e-3, (3, n))
            dev = lambda a, t=torch.float64: torch.as_tensor(a, dtype=t, device="cuda:0")
            t = dict(x=dev(x), y=dev(y), xp=dev(x), yp=dev(y), ux=dev(u[0]), uy=dev(u[1]),
                     uz=dev(u[2]), qm=dev(np.full(n, cfg.qm)),
                     id=dev(np.arange(n), torch.int32),
                     status=torch.zeros(n, dtype=torch.uint8, device="cuda:0"))
            run.push(t, 1, kernel=1, sort_every=1, tile=tile)
            key = (np.floor(y / cfg.dy).astype(np.int64) // tile) * -(-nx // tile) \
                + np.floor(x / cfg.dx).astype(np.int64) // tile
            want = np.argsort(key, kind="stable")
            assert np.array_equal(t["id"].cpu().numpy(), want), (n, spread)
            assert np.array_equal(t["xp"].cpu().numpy(), x[want]), (n, spread)
            assert np.array_equal(t["yp"].cpu().numpy(), y[want]), (n, spread)
    finally:
        run.close()
