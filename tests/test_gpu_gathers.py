"""The two gathers that FP32 maps of more than 8 channels take besides the
8 x 8-cell tiles, at the edges of their ranges: independent waves (channel
groups of 64, 128 and 256 cut short, rows read four channels or one at a
time, one or four waves to a cell block, flags) and 16 x 16-cell blocks
(ragged blocks and slabs, flags, values that BF16 pieces cannot hold).
Bounds against the FP64 oracle are the FP32 form's: 1e-5 per channel, W to
1e-6 (1e-5 for the flagged form's FP32 weight sums); the few-channel gather
(FP64 sums) is held to the same bound where it stands in for the oracle."""
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


def _device_rows(spec, shift):
    """Contiguous device rows that start `shift` floats past an aligned address."""
    buf = torch.empty(spec.numel() + shift, dtype=torch.float32, device=DEV)
    rows = buf[shift:].view(spec.shape)
    rows.copy_(spec)
    return rows


def _flagged(spec, seed):
    g = np.random.default_rng(seed)
    s = spec.numpy().copy()
    m = g.random(s.shape) < 0.05
    s[m] = g.choice([np.nan, np.inf, -np.inf], size=int(m.sum()))
    return torch.from_numpy(s)


def _cells_lonlat(g, cells):
    iy, ix = np.divmod(cells, g.nx)
    return (g.lon0 + (ix - (g.nx - 1) / 2) * g.dlon, g.lat0 + (iy - (g.ny - 1) / 2) * g.dlat)


# (n, C, nx, ny, cell', FWHM', floats past an aligned address)
WAVE = [(300, 9, 5, 3, 1.0, 3.0, 0), (4000, 16, 21, 14, 1.0, 3.0, 0),
        (4000, 64, 21, 14, 1.0, 3.0, 1), (9000, 65, 33, 17, 0.8, 3.0, 0),
        (30_000, 64, 270, 259, 0.8, 3.0, 0), (30_000, 61, 270, 259, 0.8, 3.0, 0),
        (30_000, 128, 270, 262, 0.8, 3.0, 0), (9000, 129, 33, 17, 0.8, 3.0, 0),
        (20_000, 516, 190, 175, 1.2, 3.0, 0), (20_000, 260, 270, 250, 1.2, 3.0, 2),
        (6000, 72, 25, 26, 8.0, 30.0, 0)]


@pytest.mark.parametrize("n,nchan,nx,ny,cell,fwhm,shift", WAVE)
@pytest.mark.parametrize("flags", [False, True])
def test_independent_waves_match_the_oracle(n, nchan, nx, ny, cell, fwhm, shift, flags):
    w = synth.small_cube(n=n, nchan=nchan, nx=nx, ny=ny, cell_arcmin=cell, fwhm_arcmin=fwhm,
                         seed=2600 + nchan + nx)
    spec = _flagged(w.spectra, 2601) if flags else w.spectra
    plan = hcg.hcg_plan(w.lon.to(DEV), w.lat.to(DEV), w.grid, w.fwhm_deg, w.support_deg)
    rows = _device_rows(spec, shift)
    cube = torch.full((nchan, ny, nx), 12345.0, device=DEV)
    W = torch.full((nchan, ny, nx) if flags else (ny, nx), -1.0, device=DEV)
    print(f"waves n={n} C={nchan} {nx}x{ny} flags={flags}", flush=True)
    if flags:
        hcg.hcg_grid_masked(plan, rows, cube, W)
        bare = torch.full_like(cube, 54321.0)
        hcg.hcg_grid_masked(plan, rows, bare, None)  # without the channels' weights
        torch.cuda.synchronize()
        assert torch.equal(cube.view(torch.int32), bare.view(torch.int32))
    else:
        hcg.hcg_grid(plan, rows, cube, W)
        torch.cuda.synchronize()
    cells = np.concatenate(sample_cells(w.grid, seed=5, patches=4, patch=min(6, ny, nx)))
    cl, cb = _cells_lonlat(w.grid, cells)
    V, Wr, _ = oracle.grid_points(w.lon.numpy(), w.lat.numpy(), spec.numpy(), cl, cb,
                                  w.support_deg, oracle.Kernel.gauss(w.fwhm_deg), masked=flags)
    idx = torch.from_numpy(cells).to(DEV)
    Vg = cube.reshape(nchan, -1)[:, idx].cpu().numpy()
    Wg = W.reshape(-1, nx * ny)[:, idx].cpu().numpy()
    assert_cube_close(Vg, V.T, 1e-5, f"C={nchan} {nx}x{ny}")
    assert_weights_close(Wg, np.asarray(Wr).T if flags else np.asarray(Wr)[None],
                         rtol=1e-5 if flags else 1e-6)
    plan.destroy()


@pytest.mark.parametrize("n,nchan", [(20_000, 12), (2_000_000, 129)])
def test_flagged_form_without_channel_weights(n, nchan):
    """The waves' and the blocks' flagged kernels and a spectra size on either
    side of the caches; no array for the channels' weights."""
    w = synth.small_cube(n=n // 10, nchan=1, nx=260, ny=250, cell_arcmin=0.5, seed=2700)
    g = torch.Generator().manual_seed(2701)
    lon = w.lon.repeat(10) + torch.randn(n, generator=g, dtype=torch.float64) * 1e-3
    lat = w.lat.repeat(10) + torch.randn(n, generator=g, dtype=torch.float64) * 1e-3
    plan = hcg.hcg_plan(lon.to(DEV), lat.to(DEV), w.grid, w.fwhm_deg, w.support_deg)
    gd = torch.Generator(device=DEV).manual_seed(2702)
    spec = torch.randn((n, nchan), generator=gd, device=DEV) + 3.0
    spec[torch.rand((n, nchan), generator=gd, device=DEV) < 0.05] = float("nan")
    cube = torch.empty((nchan, 250, 260), device=DEV)
    bare = torch.empty_like(cube)
    W = torch.empty_like(cube)
    print(f"flags n={n} C={nchan}", flush=True)
    hcg.hcg_grid_masked(plan, spec, cube, W)
    hcg.hcg_grid_masked(plan, spec, bare, None)
    torch.cuda.synchronize()
    assert torch.equal(cube.view(torch.int32), bare.view(torch.int32))
    for c in (0, nchan // 2, nchan - 1):  # one channel at a time: FP64 sums
        one = torch.empty((1, 250, 260), device=DEV)
        W1 = torch.empty_like(one)
        hcg.hcg_grid_masked(plan, spec[:, c:c + 1].contiguous(), one, W1)
        assert_cube_close(cube[c:c + 1].cpu().numpy(), one.cpu().numpy(), 1e-5, f"channel {c}")
        assert_weights_close(W[c].cpu().numpy(), W1[0].cpu().numpy(), rtol=1e-5)
    plan.destroy()


# dense maps whose spectra outgrow the caches: ragged blocks, a slab cut short
# (one channel, an odd count, rows that are not 8-byte aligned)
BLOCK = [(60_000, 513, 261, 253, 0.14, 0), (60_000, 514, 257, 256, 0.14, 0),
         (60_000, 512, 250, 271, 0.14, 1)]


@pytest.mark.parametrize("n,nchan,nx,ny,cell,shift", BLOCK)
def test_blocks_match_the_oracle(n, nchan, nx, ny, cell, shift):
    w = synth.small_cube(n=n, nchan=nchan, nx=nx, ny=ny, cell_arcmin=cell, seed=2800 + nchan)
    plan = hcg.hcg_plan(w.lon.to(DEV), w.lat.to(DEV), w.grid, w.fwhm_deg, w.support_deg)
    rows = _device_rows(w.spectra, shift)
    cube = torch.full((nchan, ny, nx), 12345.0, device=DEV)
    W = torch.full((ny, nx), -1.0, device=DEV)
    print(f"blocks n={n} C={nchan} {nx}x{ny}", flush=True)
    hcg.hcg_grid(plan, rows, cube, W)
    torch.cuda.synchronize()
    groups = sample_cells(w.grid, seed=6, patches=4, patch=5)
    ref = [sampled_oracle(w, c) for c in groups]
    V, Wg = gather_cells(cube, W, np.concatenate(groups))
    assert_cube_close(V.T, np.concatenate([v for v, _ in ref]).T, 1e-5, f"C={nchan}")
    assert_weights_close(Wg, np.concatenate([x for _, x in ref]))

    # values that are not finite, or that rounding to BF16 would overflow:
    # the cells within R of them, and those alone (the few-channel gather's rule)
    chans = [0, 1, 2, 3, nchan - 1]
    top = torch.finfo(torch.float32).max
    plants = [(0, 0, float("inf")), (0, n // 3, float("-inf")), (1, n // 2, float("nan")),
              (2, n // 4, top), (2, n // 5, -top), (3, 7, 1e-40), (3, 8, -float("inf")),
              (nchan - 1, n - 1, float("inf")), (nchan - 1, n - 2, float("nan"))]
    for c, s, v in plants:
        rows[s, c] = v
    hcg.hcg_grid(plan, rows, cube, W)
    few = torch.empty((len(chans), ny, nx), device=DEV)
    hcg.hcg_grid(plan, rows[:, chans].contiguous(), few, W)
    torch.cuda.synchronize()
    for k, c in enumerate(chans):
        got, want = cube[c].cpu().numpy(), few[k].cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(want)), c
        inf = np.isinf(want)
        assert np.array_equal(np.isinf(got), inf) and np.array_equal(got[inf], want[inf]), c
        ok = np.isfinite(want)
        scale = np.abs(want[ok].astype(np.float64)).max()
        assert np.abs(got[ok].astype(np.float64) - want[ok]).max() <= 1e-5 * scale, c
    others = [c for c in range(nchan) if c not in chans]
    assert bool(torch.isfinite(cube[others]).all())
    plan.destroy()


@pytest.mark.parametrize("launch", ["persistent", "items"])
def test_a_block_field_of_a_batch_equals_its_single_call(launch):
    ws = [synth.small_cube(n=n, nchan=c, nx=nx, ny=ny, cell_arcmin=0.14, seed=2900 + c)
          for n, c, nx, ny in ((60_000, 514, 261, 253), (5000, 70, 40, 33), (60_000, 513, 250, 264))]
    plan_of = lambda w: (w.lon.to(DEV), w.lat.to(DEV), w.grid, w.fwhm_deg, w.support_deg)  # noqa: E731
    batch = hcg.hcg_plan_batch([plan_of(w) for w in ws], launch=launch)
    spectra = [w.spectra.to(DEV).contiguous() for w in ws]
    cubes = [torch.full((w.nchan, w.grid.ny, w.grid.nx), -7.0, device=DEV) for w in ws]
    wts = [torch.full((w.grid.ny, w.grid.nx), -7.0, device=DEV) for w in ws]
    print(f"batch of blocks {launch}", flush=True)
    hcg.hcg_grid_batch(batch, spectra, cubes, wts)
    torch.cuda.synchronize()
    for w, s, cube, W in zip(ws, spectra, cubes, wts):
        plan = hcg.hcg_plan(*plan_of(w))
        one, W1 = torch.empty_like(cube), torch.empty_like(W)
        hcg.hcg_grid(plan, s, one, W1)
        torch.cuda.synchronize()
        assert torch.equal(one.view(torch.int32), cube.view(torch.int32))
        assert torch.equal(W1.view(torch.int32), W.view(torch.int32))
        plan.destroy()
