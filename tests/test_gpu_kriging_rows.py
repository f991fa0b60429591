"""GPU parity of the kriging form that keeps the weights of two row offsets
(destination rows at the source's spacing or half of it) against the FP64
oracle, where it can go wrong: sources of the least size, grids cut inside a
wave and inside a block's rows, rows beyond both ends of the source (offsets of
their own), columns at another ratio (source rectangles up to and beyond the
staged size), spacings that are no dyadic fraction, holes, the series form.

Bar (the definition's): NaN masks exact, values within 1e-5 relative."""
import numpy as np
import pytest
import torch

from gen import GridSpec, dem_on_grid

pytestmark = pytest.mark.gpu

REL = 1e-5


@pytest.mark.parametrize("snx,sny,h,ry,rx,shift,dnx,dny,rng,hole", [
    (5, 5, 4.0, 0.5, 0.5, 0.0, 10, 10, 3.0, 0.0),
    (40, 37, 4.0, 0.5, 0.5, 0.0, 80, 74, 3.0, 0.01),
    (300, 70, 4.0, 1.0, 1.0, 0.5, 300, 69, 3.0, 0.002),     # infill between rows
    (300, 70, 4.0, 1.0, 1.0, -6.25, 257, 85, 3.0, 0.002),   # rows beyond both ends
    (90, 600, 0.7, 0.5, 0.437, 0.0, 193, 1200, 3.0, 0.01),  # no dyadic spacing
    (90, 600, 3.3, 1.0, 1.0, 0.5, 90, 599, 3.0, 0.01),
    (900, 40, 2.0, 0.5, 3.1, 0.0, 290, 80, 3.0, 0.005),     # wide rectangles
    (2000, 30, 2.0, 1.0, 7.5, 0.25, 266, 30, 3.0, 0.005),   # beyond the staged size
    (64, 64, 4.0, 0.5, 0.5, 0.0, 128, 128, 100.0, 0.01),    # series form
])
def test_kriging_two_offsets(orc, snx, sny, h, ry, rx, shift, dnx, dny, rng, hole):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(10.0, -20.0, h, h, snx, sny)
    d = GridSpec(10.0, -20.0 + shift * h, h * rx, h * ry, dnx, dny)
    z = dem_on_grid(g, seed=7).astype(np.float32)
    z[np.random.default_rng(snx + sny).random(z.shape) < hole] = np.nan
    dst = torch.full((dny, dnx), -7.0, dtype=torch.float32, device="cuda")
    ag.auv_resample_kriging(torch.from_numpy(z).cuda(), g, dst, d, rng * h)
    torch.cuda.synchronize()
    want = orc.kriging(orc.Grid(g.x0, g.y0, g.dx, g.dy, snx, sny), z.astype(np.float64),
                       orc.Grid(d.x0, d.y0, d.dx, d.dy, dnx, dny), rng * h)
    got = dst.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = ~np.isnan(want)
    assert (np.abs(got[ok] - want[ok]) / np.abs(want[ok])).max() <= REL
