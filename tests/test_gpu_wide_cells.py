"""Maps whose cells lie far apart: columns tens of degrees wide, and centres
scattered over the sphere in no order, so that a block of neighbouring cells
has members more than 90 degrees from its middle.  The gathers of more than
eight channels against the FP64 oracle, the FP32 form's bounds: 1e-5 per
channel, W to 1e-6 (1e-5 for the flagged form's FP32 weight sums)."""
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

    def centres(self):
        lon = self.lon0 + (np.arange(self.nx) - 0.5 * (self.nx - 1)) * self.dlon
        lat = self.lat0 + (np.arange(self.ny) - 0.5 * (self.ny - 1)) * self.dlat
        cl, cb = np.meshgrid(lon, lat)
        return cl.ravel(), cb.ravel()


def _samples_near(cl, cb, n, reach, seed):
    """n samples within about `reach` degrees of cells chosen at random."""
    g = np.random.default_rng(seed)
    k = g.integers(0, len(cl), n)
    lat = np.clip(cb[k] + g.uniform(-reach, reach, n), -89.9, 89.9)
    lon = cl[k] + g.uniform(-reach, reach, n) / np.cos(np.radians(lat))
    return lon, lat


def _spectra(n, nchan, flags, seed):
    g = np.random.default_rng(seed)
    s = (g.standard_normal((n, nchan)) + 2.0).astype(np.float32)
    if flags:
        s[g.random(s.shape) < 0.05] = np.nan
    return s


def _check(cube, W, lon, lat, spec, cl, cb, support, kernel, flags, cells=None, what=""):
    cells = np.arange(len(cl)) if cells is None else cells
    V, Wr, npair = oracle.grid_points(lon, lat, spec, cl[cells], cb[cells], support, kernel,
                                      masked=flags)
    assert int(np.max(npair)) > 0
    idx = torch.from_numpy(cells).to(DEV)
    Vg = cube.reshape(cube.shape[0], -1)[:, idx].cpu().numpy()
    Wg = W.reshape(-1, len(cl))[:, idx].cpu().numpy()
    assert_cube_close(Vg, V.T, 1e-5, what)
    assert_weights_close(Wg, np.asarray(Wr).T if flags else np.asarray(Wr)[None],
                         rtol=1e-5 if flags else 1e-6)


def _grid(plan, spec, flags, nchan, ny, nx):
    cube = torch.full((nchan, ny, nx), 12345.0, device=DEV)
    W = torch.full((nchan, ny, nx) if flags else (ny, nx), -1.0, device=DEV)
    (hcg.hcg_grid_masked if flags else hcg.hcg_grid)(plan, torch.from_numpy(spec).to(DEV), cube, W)
    torch.cuda.synchronize()
    return cube, W


# (FWHM, support, row step) in degrees: a narrow and a wide support
@pytest.mark.parametrize("fwhm,support,dlat", [(0.4, 0.5, 0.05), (1.2, 1.5, 0.3)])
@pytest.mark.parametrize("nchan", [11, 12])
@pytest.mark.parametrize("flags", [False, True])
def test_columns_seventy_degrees_apart(fwhm, support, dlat, nchan, flags):
    g = Grid(4, 6, 10.0, 3.0, 70.0, dlat)
    cl, cb = g.centres()
    lon, lat = _samples_near(cl, cb, 700, support, 41)
    spec = _spectra(700, nchan, flags, 42)
    field = (torch.from_numpy(lon).to(DEV), torch.from_numpy(lat).to(DEV), g, fwhm, support)
    plan = hcg.hcg_plan(*field)
    print(f"columns fwhm={fwhm} C={nchan} flags={flags}", flush=True)
    cube, W = _grid(plan, spec, flags, nchan, g.ny, g.nx)
    kern = oracle.Kernel.gauss(fwhm)
    _check(cube, W, lon, lat, spec, cl, cb, support, kern, flags, what="single")
    plan.destroy()
    if not flags:
        for launch in ("persistent", "items"):
            batch = hcg.hcg_plan_batch([field], launch=launch)
            cube.fill_(12345.0)
            W.fill_(-1.0)
            hcg.hcg_grid_batch(batch, [torch.from_numpy(spec).to(DEV)], [cube], [W])
            torch.cuda.synchronize()
            _check(cube, W, lon, lat, spec, cl, cb, support, kern, flags, what=launch)


@pytest.mark.parametrize("flags", [False, True])
def test_blocks_of_columns_fifteen_degrees_apart(flags):
    """16 columns over 225 degrees, rows close together: dense by its area, so
    2048 channels take the 16 x 16-cell blocks."""
    g = Grid(16, 1024, 200.0, 0.0, 15.0, 7e-6)
    cl, cb = g.centres()
    n, nchan, support = 20_000, 2048, 0.5
    lon, lat = _samples_near(cl, cb, n, support, 43)
    spec = _spectra(n, nchan, flags, 44)
    plan = hcg.hcg_plan(torch.from_numpy(lon).to(DEV), torch.from_numpy(lat).to(DEV), g, 0.4, support)
    print(f"blocks of wide columns flags={flags}", flush=True)
    cube, W = _grid(plan, spec, flags, nchan, g.ny, g.nx)
    rows = np.array([0, 517, 1023])
    cells = (rows[:, None] * g.nx + np.arange(g.nx)).ravel()
    _check(cube, W, lon, lat, spec, cl, cb, support, oracle.Kernel.gauss(0.4), flags, cells)
    plan.destroy()


@pytest.mark.parametrize("kernel,support", [
    (("gauss", 3.2), 4.0), (("gauss", 0.4), 0.5), (("elliptic", 3.2, 2.0, 30.0), 4.0)])
@pytest.mark.parametrize("flags", [False, True])
def test_centres_scattered_over_the_sphere(kernel, support, flags):
    rng = np.random.default_rng(45)
    ny, nx, n, nchan = 9, 13, 3000, 20
    cl = rng.uniform(0.0, 360.0, ny * nx)
    cb = np.degrees(np.arcsin(rng.uniform(-0.98, 0.98, ny * nx)))
    lon, lat = _samples_near(cl, cb, n, support, 46)
    spec = _spectra(n, nchan, flags, 47)
    make = {"gauss": (hcg.Kernel.gauss, oracle.Kernel.gauss),
            "elliptic": (hcg.Kernel.elliptic, oracle.Kernel.elliptic)}[kernel[0]]
    plan = hcg.hcg_plan_ex(torch.from_numpy(lon).to(DEV), torch.from_numpy(lat).to(DEV),
                           make[0](*kernel[1:]), support,
                           cell_lon=torch.from_numpy(cl.reshape(ny, nx)).to(DEV),
                           cell_lat=torch.from_numpy(cb.reshape(ny, nx)).to(DEV), nside=16)
    print(f"scattered {kernel} flags={flags}", flush=True)
    cube, W = _grid(plan, spec, flags, nchan, ny, nx)
    _check(cube, W, lon, lat, spec, cl, cb, support, make[1](*kernel[1:]), flags)
    plan.destroy()


# ---------------------------------------------------------------------------
# Cells far wider apart than the support: the squared distances of a pair are
# tiny beside those to the middle of its block of cells.
# ---------------------------------------------------------------------------
POINTS = Grid(24, 20, 100.0, 0.0, 2.0, 2.0)


@pytest.mark.parametrize("nchan", [1, 2, 4, 8, 12])
@pytest.mark.parametrize("flags", [False, True])
def test_support_of_zero_takes_the_samples_on_the_cells(nchan, flags):
    """R = 0: a cell's sample, at exactly its centre, and no other; weight 1."""
    g = POINTS
    cl, cb = g.centres()
    lon, lat = _samples_near(cl, cb, 200_000, 0.9, 48)
    lon = np.concatenate([cl, lon])
    lat = np.concatenate([cb, lat])
    n = len(lon)
    spec = _spectra(n, nchan, flags, 49)
    field = (torch.from_numpy(lon).to(DEV), torch.from_numpy(lat).to(DEV), g, 0.05, 0.0)
    plan = hcg.hcg_plan(*field, nside=64)
    print(f"support 0 C={nchan} flags={flags}", flush=True)
    cube, W = _grid(plan, spec, flags, nchan, g.ny, g.nx)
    want = spec[:len(cl)].T.reshape(nchan, g.ny, g.nx)
    np.testing.assert_array_equal(cube.cpu().numpy(), want)
    np.testing.assert_array_equal(W.cpu().numpy(), np.isfinite(want).astype(np.float32)
                                  if flags else np.ones((g.ny, g.nx), np.float32))
    plan.destroy()
    if not flags:
        for launch in ("persistent", "items"):
            batch = hcg.hcg_plan_batch([field], launch=launch, nside=64)
            cube.fill_(12345.0)
            W.fill_(-1.0)
            hcg.hcg_grid_batch(batch, [torch.from_numpy(spec).to(DEV)], [cube], [W])
            np.testing.assert_array_equal(cube.cpu().numpy(), want)
            np.testing.assert_array_equal(W.cpu().numpy(), np.ones((g.ny, g.nx), np.float32))


@pytest.mark.parametrize("nchan", [1, 3, 8, 12])
@pytest.mark.parametrize("flags", [False, True])
@pytest.mark.parametrize("shape", ["gauss", "elliptic"])
def test_support_far_below_the_cells(nchan, flags, shape):
    """Cells of 2 degrees, a support of 0.02 arcsec: 3.6e5 times less."""
    g = POINTS
    cl, cb = g.centres()
    fwhm, support, n = 0.016 / 3600, 0.02 / 3600, 120_000
    lon, lat = _samples_near(cl, cb, n, 1.1 * support, 50)
    spec = _spectra(n, nchan, flags, 51)
    dev = (torch.from_numpy(lon).to(DEV), torch.from_numpy(lat).to(DEV))
    if shape == "gauss":
        plan = hcg.hcg_plan(*dev, g, fwhm, support, nside=64)
        kern = oracle.Kernel.gauss(fwhm)
    else:
        plan = hcg.hcg_plan_ex(*dev, hcg.Kernel.elliptic(fwhm, 0.7 * fwhm, 30.0), support, grid=g,
                               nside=64)
        kern = oracle.Kernel.elliptic(fwhm, 0.7 * fwhm, 30.0)
    print(f"tiny support C={nchan} flags={flags} {shape}", flush=True)
    cube, W = _grid(plan, spec, flags, nchan, g.ny, g.nx)
    cells = np.arange(0, len(cl), 7)
    _check(cube, W, lon, lat, spec, cl, cb, support, kern, flags, cells)
    plan.destroy()
