"""The 16 x 16-cell blocks split FP32 operands into BF16 pieces: spectra and
weights whose pieces fall below the smallest normal number.  Against the FP64
oracle, the FP32 form's bounds: 1e-5 per channel, W to 1e-6 (1e-5 for the
flagged form's FP32 weight sums)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2012_13173_amd as hcg
import synth
from tests.gridcheck import assert_cube_close, assert_weights_close

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _centres(g, cells):
    iy, ix = np.divmod(cells, g.nx)
    return (g.lon0 + (ix - (g.nx - 1) / 2) * g.dlon, g.lat0 + (iy - (g.ny - 1) / 2) * g.dlat)


def _run(w, spec, flags, cells, what, support=None, wtol=1e-6):
    support = w.support_deg if support is None else support
    plan = hcg.hcg_plan(w.lon.to(DEV), w.lat.to(DEV), w.grid, w.fwhm_deg, support)
    nchan, ny, nx = spec.shape[1], w.grid.ny, w.grid.nx
    cube = torch.full((nchan, ny, nx), 12345.0, device=DEV)
    W = torch.full((nchan, ny, nx) if flags else (ny, nx), -1.0, device=DEV)
    print(what, flush=True)
    (hcg.hcg_grid_masked if flags else hcg.hcg_grid)(plan, torch.from_numpy(spec).to(DEV), cube, W)
    torch.cuda.synchronize()
    plan.destroy()
    cl, cb = _centres(w.grid, cells)
    V, Wr, _ = oracle.grid_points(w.lon.numpy(), w.lat.numpy(), spec, cl, cb, support,
                                  oracle.Kernel.gauss(w.fwhm_deg), masked=flags)
    idx = torch.from_numpy(cells).to(DEV)
    Vg = cube.reshape(nchan, -1)[:, idx].cpu().numpy()
    Wg = W.reshape(-1, nx * ny)[:, idx].cpu().numpy()
    # a result is rounded to a multiple of 2^-149: up to 2^-150 beside the bound
    rms = np.sqrt(np.nanmean(V ** 2, axis=0))
    e = assert_cube_close(Vg, V.T, 1e-5 + 2.0 ** -150 / rms[rms > 0].min(), what)
    print(f"{what}: largest per-channel error {e.max():.2e}", flush=True)
    assert_weights_close(Wg, np.asarray(Wr).T if flags else np.asarray(Wr)[None],
                         rtol=1e-5 if flags else wtol)
    return cube


# 1.2e-38 is the smallest normal float, 9.2e-41 the smallest BF16
@pytest.mark.parametrize("scale", [1e-30, 1e-34, 1e-36, 1e-38, 1e-41])
@pytest.mark.parametrize("flags", [False, True])
def test_spectra_of_small_values(scale, flags):
    w = synth.small_cube(n=60_000, nchan=513, nx=261, ny=253, cell_arcmin=0.14, seed=3001)
    spec = (w.spectra.numpy().astype(np.float64) * scale).astype(np.float32)
    if flags:
        spec[np.random.default_rng(3002).random(spec.shape) < 0.05] = np.nan
    cells = np.random.default_rng(3003).choice(261 * 253, 60, replace=False)
    _run(w, spec, flags, cells, f"values of {scale:g} flags={flags}")


@pytest.mark.parametrize("flags", [False, True])
def test_small_values_beside_large_zero_and_non_finite_ones(flags):
    """In one block and slab: channels of tiny, of zero and of ordinary values,
    a channel that is tiny on one side of the map and large on the other, one
    that is zero there, and a non-finite sample among tiny ones."""
    w = synth.small_cube(n=60_000, nchan=513, nx=261, ny=253, cell_arcmin=0.14, seed=3004)
    spec = w.spectra.numpy().astype(np.float32).copy()
    west = w.lon.numpy() < np.median(w.lon.numpy())
    spec[:, 1] *= np.float32(1e-36)
    spec[:, 2] = 0.0
    spec[west, 3] *= np.float32(1e-36)
    spec[~west, 3] *= np.float32(1e30)
    spec[:, 4] *= np.float32(1e-35)
    spec[west, 4] = 0.0
    spec[:, 5] *= np.float32(1e-36)
    if flags:
        spec[100, 5] = np.inf
    cells = np.random.default_rng(3005).choice(261 * 253, 60, replace=False)
    cube = _run(w, spec, flags, cells, f"mixed values flags={flags}").cpu().numpy()
    assert not cube[2][np.isfinite(cube[2])].any()
    # channel 3 cell by cell (its norm sees the large side alone)
    cl, cb = _centres(w.grid, cells)
    V, _, _ = oracle.grid_points(w.lon.numpy(), w.lat.numpy(), spec[:, 3:5], cl, cb, w.support_deg,
                                 oracle.Kernel.gauss(w.fwhm_deg))
    for k in (0, 1):
        got = cube[3 + k].reshape(-1)[cells].astype(np.float64)
        tiny = np.abs(V[:, k]) < 1e-30
        assert tiny.sum() > 5
        rms = np.sqrt(np.mean(V[tiny, k] ** 2))
        assert np.abs(got - V[:, k])[tiny].max() <= 1e-4 * rms  # 10 times 1e-5, as every cell
    if not flags:  # non-finite values among tiny ones: the few-channel gather's rule
        rows = torch.from_numpy(spec).to(DEV)
        for s, v in ((100, np.inf), (40_000, -np.inf), (70, np.nan)):
            rows[s, 5] = float(v)
        plan = hcg.hcg_plan(w.lon.to(DEV), w.lat.to(DEV), w.grid, w.fwhm_deg, w.support_deg)
        many = torch.empty((513, 253, 261), device=DEV)
        one = torch.empty((1, 253, 261), device=DEV)
        hcg.hcg_grid(plan, rows, many)
        hcg.hcg_grid(plan, rows[:, 5:6].contiguous(), one)
        torch.cuda.synchronize()
        a, b = many[5].cpu().numpy(), one[0].cpu().numpy()
        assert np.array_equal(np.isnan(a), np.isnan(b))
        assert np.array_equal(np.isinf(a), np.isinf(b)) and np.isinf(b).any()
        ok = np.isfinite(b)
        assert np.abs(a[ok].astype(np.float64) - b[ok]).max() <= 1e-4 * np.abs(b[ok]).max()
        plan.destroy()


@pytest.mark.parametrize("flags", [False, True])
def test_cells_that_only_far_samples_reach(flags):
    """A support of 13.1 sigma and samples on one side of the map: cells whose
    samples all weigh 2^-116 to 2^-124 (whose exponents, rounded to FP32, are
    off by up to 2^-18: the weights by 2.6e-6)."""
    w = synth.small_cube(n=60_000, nchan=513, nx=270, ny=253, cell_arcmin=0.14, seed=3006)
    g = w.grid
    sigma = w.fwhm_deg / 2.3548200450309493
    support = 13.1 * sigma
    edge = g.lon0 - 0.06
    # squeeze the samples into the first columns
    lon = w.lon.numpy()
    first = g.lon0 - 0.5 * (g.nx - 1) * g.dlon
    span = (lon - lon.min()) / (lon.max() - lon.min())
    w.lon = torch.from_numpy(first + span * (edge - first))
    spec = w.spectra.numpy().astype(np.float32).copy()
    if flags:
        spec[np.random.default_rng(3007).random(spec.shape) < 0.05] = np.nan
    cl, cb = _centres(g, np.arange(g.nx * g.ny))
    gap = (cl - edge) * np.cos(np.radians(cb))
    cells = np.nonzero((gap > 12.7 * sigma) & (gap < 13.05 * sigma))[0]
    cells = np.random.default_rng(3008).choice(cells, 50, replace=False)
    _run(w, spec, flags, cells, f"far samples flags={flags}", support, wtol=3e-6)
