"""Calls of more work-items than one dimension of a launch holds (2^32)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2012_13173_amd as hcg
from tests.gridcheck import assert_cube_close, assert_weights_close

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


class Grid:
    def __init__(self, nx, ny, lon0, lat0, dlon, dlat):
        self.nx, self.ny, self.lon0, self.lat0, self.dlon, self.dlat = nx, ny, lon0, lat0, dlon, dlat


def _need(gib):
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < gib * 2 ** 30:
        pytest.skip(f"needs {gib} GiB of device memory")


@pytest.fixture(autouse=True)
def _give_back():
    yield
    torch.cuda.empty_cache()


def test_few_channels_of_2_to_the_32_values():
    """2^29 samples of eight channels: the values put into the plan's order
    first are the ones read through its permutation."""
    _need(120)
    n, nchan = 1 << 29, 8
    g = Grid(21, 13, 50.0, 20.0, 0.3, 0.3)
    gen = torch.Generator(device=DEV).manual_seed(61)
    lon = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) * 6.6 + 46.7
    lat = torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) * 4.2 + 17.9
    plan = hcg.hcg_plan(lon, lat, g, 0.1, 0.12)
    spec = torch.empty((n, nchan), device=DEV)
    for c in range(nchan):
        spec[:, c] = (lon * (c + 1)).sin()
    del lon, lat
    cube = torch.full((nchan, g.ny, g.nx), 12345.0, device=DEV)
    W = torch.full((g.ny, g.nx), -1.0, device=DEV)
    cube_p, W_p = torch.empty_like(cube), torch.empty_like(W)
    print("2^32 values", flush=True)
    hcg.hcg_grid(plan, spec, cube, W)
    hcg.hcg_grid_noalloc(plan, spec, cube_p, W_p)
    torch.cuda.synchronize()
    plan.destroy()
    assert torch.equal(cube.view(torch.int32), cube_p.view(torch.int32))
    assert torch.equal(W.view(torch.int32), W_p.view(torch.int32))
    # many thousand samples a cell: the mean of a smooth function of longitude
    lon_c = g.lon0 + (torch.arange(g.nx, dtype=torch.float64) - 0.5 * (g.nx - 1)) * g.dlon
    for c in range(nchan):
        want = (lon_c * (c + 1)).sin()[None, :].expand(g.ny, g.nx)
        assert (cube[c].cpu().double() - want).abs().max() < 0.2


@pytest.mark.parametrize("side,n,nchan,batch", [(16384, 1700, 8, False), (32768, 420, 1, False),
                                                (32768, 420, 1, True)])
def test_few_channels_of_many_tiles(side, n, nchan, batch):
    """4.2M tiles of four workgroups and 16.8M of one, every sample a candidate
    of every tile (few enough to keep the test short, too many for one wave)."""
    _need(130)
    step = 0.25 / side
    g = Grid(side, side, 120.0, 10.0, step, step)
    rng = np.random.default_rng(62)
    lon, lat = 120.0 + rng.uniform(-0.02, 0.02, n), 10.0 + rng.uniform(-0.02, 0.02, n)
    spec = (rng.standard_normal((n, nchan)) + 2.0).astype(np.float32)
    fwhm, support = 0.3, 0.3
    dev = (torch.from_numpy(lon).to(DEV), torch.from_numpy(lat).to(DEV))
    rows = torch.from_numpy(spec).to(DEV)
    cube = torch.full((nchan, side, side), 12345.0, device=DEV)
    W = torch.full((side, side), -1.0, device=DEV)
    print(f"{side} x {side} C={nchan} batch={batch}", flush=True)
    if batch:
        b = hcg.hcg_plan_batch([(*dev, g, fwhm, support)], launch="items", nside=64)
        hcg.hcg_grid_batch(b, [rows], [cube], [W])
    else:
        b = hcg.hcg_plan(*dev, g, fwhm, support, nside=64)
        hcg.hcg_grid(b, rows, cube, W)
    torch.cuda.synchronize()
    b.destroy()
    cells = np.concatenate([[0, side - 1, side * side - 1, side * (side - 1)],
                            rng.integers(0, side * side, 60)])
    iy, ix = np.divmod(cells, side)
    cl = g.lon0 + (ix - 0.5 * (side - 1)) * g.dlon
    cb = g.lat0 + (iy - 0.5 * (side - 1)) * g.dlat
    V, Wr, _ = oracle.grid_points(lon, lat, spec, cl, cb, support, oracle.Kernel.gauss(fwhm))
    idx = torch.from_numpy(cells).to(DEV)
    assert_cube_close(cube.reshape(nchan, -1)[:, idx].cpu().numpy(), V.T, 1e-5, f"{side}")
    assert_weights_close(W.reshape(-1)[idx].cpu().numpy(), Wr)
    # and no cell left out
    assert not bool((W < 0).any()) and not bool((cube == 12345.0).any())


@pytest.mark.parametrize("nchan", [2 ** 29 + 4, 2 ** 28 + 3])
@pytest.mark.parametrize("launch", [None, "items", "persistent"])
def test_one_cell_of_half_a_billion_channels(nchan, launch):
    """2^24 workgroups and byte offsets past 2^31 within a row, rows read four
    channels or one at a time: one sample, so V is the sample's spectrum."""
    _need(12)
    g = Grid(1, 1, 30.0, 40.0, 0.01, 0.01)
    field = (torch.tensor([30.001], dtype=torch.float64, device=DEV),
             torch.tensor([40.001], dtype=torch.float64, device=DEV), g, 0.05, 0.06)
    plan = hcg.hcg_plan_batch([field], launch=launch) if launch else hcg.hcg_plan(*field)
    spec = torch.empty((1, nchan), device=DEV)
    spec.uniform_(1.0, 2.0, generator=torch.Generator(device=DEV).manual_seed(63))
    cube = torch.full((nchan, 1, 1), 12345.0, device=DEV)
    print(f"one cell C={nchan} {launch}", flush=True)
    if launch:
        hcg.hcg_grid_batch(plan, [spec], [cube])
    else:
        hcg.hcg_grid(plan, spec, cube)
    torch.cuda.synchronize()
    plan.destroy()
    # w s / w: a product and a quotient rounded, the reciprocal too
    worst = float((cube.view(-1) - spec.view(-1)).abs_().max())
    assert worst <= 4 * 2.0 ** -23
