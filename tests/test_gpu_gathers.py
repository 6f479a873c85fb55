"""The gathers of FP32 maps of more than 8 channels at the edges of their
ranges.  The few-channel gather (FP64 sums) stands in for the oracle: 1e-5 per
channel, W of the flagged form (FP32 sums) to 1e-5."""
import pytest
import torch

import paper_2012_13173_amd as hcg
import synth
from tests.gridcheck import assert_cube_close, assert_weights_close

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


@pytest.mark.parametrize("n,nchan", [(20_000, 12), (2_000_000, 129)])
def test_flagged_form_without_channel_weights(n, nchan):
    """No array for the channels' weights; spectra on either side of the caches."""
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
