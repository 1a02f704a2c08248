"""The cell sort with buckets of more particles than one workgroup sorts (16384;
parts of 8192 above): around both counts, all particles in one tile, half of
them, a row of tiles, two buckets.  The order is the stable order by tile,
exactly; a tiled push in place over it gives every particle its step, bit for
bit that of the cache-served kernel (so the tiles' starts are right)."""
import numpy as np
import pytest
import torch

from gpu_util import GpuRun, log
from workloads import make_config

pytestmark = pytest.mark.gpu

# (nx, ny, tile): 272 tiles (buckets of 2), 3072 (16), 41616 (256)
GRIDS = [(136, 128, 8), (512, 384, 8), (816, 816, 4)]
CROWDS = {"one tile": (16384, 16385, 24576, 24577, 200001), "half": (32768, 32770, 1048576),
          "row": (100000, 700000), "two buckets": (33000, 131072)}


def crowd(kind, n, tile, cfg, rng):
    x, y = rng.uniform(0, cfg.Lx, n), rng.uniform(0, cfg.Ly, n)
    if kind == "row":
        return x, 5 * tile + y % tile
    if kind == "two buckets":
        far = rng.uniform(0, 1, n) < 0.5
        return x % tile, np.where(far, cfg.Ly - tile + y % tile, y % tile)
    gathered = np.ones(n, bool) if kind == "one tile" else rng.uniform(0, 1, n) < 0.5
    return (np.where(gathered, 3 * tile + x % tile, x),
            np.where(gathered, 7 * tile + y % tile, y))


@pytest.mark.parametrize("nx,ny,tile", GRIDS)
@pytest.mark.parametrize("kind", CROWDS)
def test_crowded_buckets(nx, ny, tile, kind):
    cfg = make_config("harris64", nx=nx, ny=ny)
    run = GpuRun(cfg, cfg.fields())
    rng = np.random.default_rng(nx + tile)
    dev = lambda a, t=torch.float64: torch.as_tensor(a, dtype=t, device="cuda:0")
    try:
        for n in CROWDS[kind]:
            log(f"{nx}x{ny} tile {tile}: {n} {kind}")
            x, y = crowd(kind, n, tile, cfg, rng)
            u = rng.normal(0, 1e-3, (3, n))

            def state():
                return dict(x=dev(x), y=dev(y), xp=dev(x), yp=dev(y), ux=dev(u[0]), uy=dev(u[1]),
                            uz=dev(u[2]), qm=dev(np.full(n, cfg.qm)),
                            id=dev(np.arange(n), torch.int32),
                            status=torch.zeros(n, dtype=torch.uint8, device="cuda:0"))
            t = state()
            run.push(t, 1, kernel=1, sort_every=1, tile=tile)
            key = (np.floor(y).astype(np.int64) // tile) * -(-nx // tile) \
                + np.floor(x).astype(np.int64) // tile
            want = np.argsort(key, kind="stable")
            assert np.array_equal(t["id"].cpu().numpy(), want), n
            plain, tiled = state(), state()
            run.push(plain, 1, kernel=1)
            run.push(tiled, 1, kernel=2, sort_every=1, tile=tile, keep_order=1)
            for k in ("x", "y", "xp", "yp", "ux", "uy", "uz"):
                assert torch.equal(plain[k], tiled[k]), (n, k)
    finally:
        run.close()
