"""The few-channel gather (FP32, C <= 8): every channel-count kernel, at the
numbers of waves per sub-block of cells that the launch chooses from (one,
four, and as many as a workgroup takes), with the values read through the
permutation and put into the plan's order first, against the oracle on
sampled cells: 1e-5 per channel, W to 1e-6 (the FP32 form's bounds; both
sides sum in FP64 and differ by the rounding of the weights, 2.7e-7)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2012_13173_amd as hcg
import synth
from tests.gridcheck import (assert_cube_close, assert_weights_close, gather_cells, sample_cells,
                             sampled_oracle)

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

# (n, C, nx, ny, cell', FWHM', support in sigma): ragged tiles; 2 tiles;
# four waves a sub-block; one wave; n on both sides of the value sort's
# threshold; cells wider than the support; a wide support (0.64 deg)
CASES = [(400, 1, 9, 7, 1.0, 3.0, 3.0), (400, 8, 13, 3, 1.0, 3.0, 3.0),
         (30_000, 2, 190, 141, 0.5, 3.0, 3.0), (30_000, 3, 150, 141, 0.5, 3.0, 3.0),
         (262_143, 4, 170, 90, 0.5, 3.0, 3.0), (262_144, 4, 170, 90, 0.5, 3.0, 3.0),
         (300_000, 1, 40, 33, 9.0, 3.0, 3.0), (270_000, 7, 390, 280, 0.5, 2.5, 5.0),
         (20_000, 5, 33, 21, 10.0, 30.0, 3.0)]


@pytest.mark.parametrize("n,nchan,nx,ny,cell,fwhm,sigmas", CASES)
def test_few_channels_match_the_oracle(n, nchan, nx, ny, cell, fwhm, sigmas):
    w = synth.small_cube(n=n, nchan=nchan, nx=nx, ny=ny, cell_arcmin=cell, fwhm_arcmin=fwhm,
                         support_sigma=sigmas, seed=1700 + nchan + nx)
    plan = hcg.hcg_plan(w.lon.to(DEV), w.lat.to(DEV), w.grid, w.fwhm_deg, w.support_deg)
    spec = w.spectra.to(DEV).contiguous()
    shape = (nchan, ny, nx)
    maps = []
    for grid in (hcg.hcg_grid, hcg.hcg_grid_noalloc):
        cube = torch.full(shape, 12345.0, dtype=torch.float32, device=DEV)
        W = torch.full(shape[1:], -1.0, dtype=torch.float32, device=DEV)
        print(f"{grid.__name__} n={n} C={nchan} {nx}x{ny}", flush=True)
        grid(plan, spec, cube, W)
        torch.cuda.synchronize()
        maps.append((cube, W))
    (cube, W), (cube_b, W_b) = maps
    # the values' order in memory does not reach the sums
    assert torch.equal(cube.view(torch.int32), cube_b.view(torch.int32))
    assert torch.equal(W.view(torch.int32), W_b.view(torch.int32))
    groups = sample_cells(w.grid, seed=5, patches=4, patch=min(6, ny))
    cells = np.concatenate(groups)
    ref = [sampled_oracle(w, c) for c in groups]
    V, Wg = gather_cells(cube, W, cells)
    assert_cube_close(V.T, np.concatenate([v for v, _ in ref]).T, 1e-5, f"C={nchan} {nx}x{ny}")
    assert_weights_close(Wg, np.concatenate([x for _, x in ref]))
    # flags: none set, so each channel's W is the map's and V is unchanged to
    # the last place (the same sums in the same order)
    cube_m = torch.empty_like(cube)
    W_m = torch.empty_like(cube)
    hcg.hcg_grid_masked(plan, spec, cube_m, W_m)
    torch.cuda.synchronize()
    torch.testing.assert_close(cube_m, cube, rtol=2e-7, atol=0, equal_nan=True)
    torch.testing.assert_close(W_m, W[None].expand_as(W_m), rtol=2e-7, atol=0)
    plan.destroy()


# (n, C, nx, ny, cell', flags): tiles of two candidates and none; about one
# chunk of 64; more than one
LANE = [(400, 1, 203, 150, 2.0, False), (400, 7, 203, 150, 2.0, True),
        (9000, 2, 190, 141, 1.2, False), (9000, 8, 190, 141, 1.2, True),
        (26_000, 4, 262, 259, 0.9, False), (26_000, 5, 262, 259, 0.9, True)]


@pytest.mark.parametrize("n,nchan,nx,ny,cell,flags", LANE)
@pytest.mark.parametrize("fwhm", [3.0, 32.0])
def test_tiles_of_few_candidates_match_the_oracle(n, nchan, nx, ny, cell, flags, fwhm):
    """Maps whose tiles go to one wave each, alone and in a batch, against the
    oracle: the same bounds."""
    cell = cell * fwhm / 3.0
    w = synth.small_cube(n=n, nchan=nchan, nx=nx, ny=ny, cell_arcmin=cell, fwhm_arcmin=fwhm,
                         seed=1800 + nchan + nx)
    spec = w.spectra.clone()
    if flags:
        spec[torch.rand(spec.shape, generator=torch.Generator().manual_seed(3)) < 0.1] = float("nan")
    plan = hcg.hcg_plan(w.lon.to(DEV), w.lat.to(DEV), w.grid, w.fwhm_deg, w.support_deg)
    cube = torch.full((nchan, ny, nx), 12345.0, device=DEV)
    W = torch.full((nchan, ny, nx) if flags else (ny, nx), -1.0, device=DEV)
    print(f"lanes n={n} C={nchan} {nx}x{ny} fwhm={fwhm}", flush=True)
    (hcg.hcg_grid_masked if flags else hcg.hcg_grid)(plan, spec.to(DEV), cube, W)
    torch.cuda.synchronize()
    cells = np.concatenate(sample_cells(w.grid, seed=5, patches=5, patch=8))
    iy, ix = np.divmod(cells, nx)
    g = w.grid
    cl = g.lon0 + (ix - (nx - 1) / 2) * g.dlon
    cb = g.lat0 + (iy - (ny - 1) / 2) * g.dlat
    V, Wr, _ = oracle.grid_points(w.lon.numpy(), w.lat.numpy(), spec.numpy(), cl, cb,
                                  w.support_deg, oracle.Kernel.gauss(w.fwhm_deg), masked=flags)
    idx = torch.from_numpy(cells).to(DEV)
    assert_cube_close(cube.reshape(nchan, -1)[:, idx].cpu().numpy(), V.T, 1e-5, f"C={nchan}")
    assert_weights_close(W.reshape(-1, nx * ny)[:, idx].cpu().numpy(),
                         np.asarray(Wr).T if flags else np.asarray(Wr)[None])
    if not flags:
        batch = hcg.hcg_plan_batch([(w.lon.to(DEV), w.lat.to(DEV), g, w.fwhm_deg, w.support_deg)])
        cube_b, W_b = torch.empty_like(cube), torch.empty_like(W)
        hcg.hcg_grid_batch(batch, [spec.to(DEV)], [cube_b], [W_b])
        torch.cuda.synchronize()
        torch.testing.assert_close(cube_b, cube, rtol=1e-6, atol=1e-7, equal_nan=True)
        torch.testing.assert_close(W_b, W, rtol=1e-6, atol=0)


# sub-blocks of two cells (one channel: eight and sixteen) by several waves and
# by one; one wave to a tile
@pytest.mark.parametrize("n,nx,ny,cell", [(20_000, 45, 37, 0.75), (60_000, 150, 141, 0.5),
                                          (9000, 190, 141, 1.2)])
@pytest.mark.parametrize("nchan", [1, 5, 8])
@pytest.mark.parametrize("shape", ["elliptic", "tapered_sinc"])
def test_flagged_channels_of_the_other_kernel_shapes(n, nx, ny, cell, nchan, shape):
    w = synth.small_cube(n=n, nchan=nchan, nx=nx, ny=ny, cell_arcmin=cell, seed=1900 + nchan + nx)
    spec = w.spectra.clone()
    spec[torch.rand(spec.shape, generator=torch.Generator().manual_seed(4)) < 0.1] = float("inf")
    args, support = {"elliptic": ((0.05, 0.03, 25.0), 0.06),
                     "tapered_sinc": ((2.5 / 60, 3.5 / 60), 3.75 / 60)}[shape]
    plan = hcg.hcg_plan_ex(w.lon.to(DEV), w.lat.to(DEV), getattr(hcg.Kernel, shape)(*args), support,
                           grid=w.grid)
    cube = torch.full((nchan, ny, nx), 12345.0, device=DEV)
    W = torch.full((nchan, ny, nx), -1.0, device=DEV)
    print(f"{shape} n={n} C={nchan} {nx}x{ny}", flush=True)
    hcg.hcg_grid_masked(plan, spec.to(DEV), cube, W)
    torch.cuda.synchronize()
    plan.destroy()
    g = w.grid
    cells = np.concatenate(sample_cells(g, seed=8, patches=4, patch=6))
    iy, ix = np.divmod(cells, nx)
    V, Wr, _ = oracle.grid_points(w.lon.numpy(), w.lat.numpy(), spec.numpy(),
                                  g.lon0 + (ix - (nx - 1) / 2) * g.dlon,
                                  g.lat0 + (iy - (ny - 1) / 2) * g.dlat, support,
                                  getattr(oracle.Kernel, shape)(*args), masked=True)
    idx = torch.from_numpy(cells).to(DEV)
    Vg = cube.reshape(nchan, -1)[:, idx].cpu().numpy()
    Wg = W.reshape(nchan, -1)[:, idx].cpu().numpy()
    assert_cube_close(Vg, V.T, 1e-5, f"{shape} C={nchan}")
    # (a sinc's weights change sign: a sum's error is one of the weights')
    Wr = np.asarray(Wr).T
    np.testing.assert_allclose(Wg, Wr, rtol=1e-6, atol=1e-6 * np.abs(Wr).max())
