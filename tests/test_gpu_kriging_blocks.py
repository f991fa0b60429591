"""GPU parity of kriging where the kept-weights form's source rectangle decides the
rows per block or hands the grid to the general form: columns 2.4 to 8 times
coarser than the source's, rows at its spacing and half of it, enough blocks for
32 and 64 rows each.  Against the FP64 oracle: NaN masks exact, values within
1e-5 relative."""
import numpy as np
import pytest
import torch

from gen import GridSpec, dem_on_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ry", [1.0, 0.5])
@pytest.mark.parametrize("rx", [2.4, 3.0, 3.1, 8.0])
def test_wide_rectangles(orc, rx, ry):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    snx, sny = 1200, int(1100 * ry)
    g = GridSpec(0.0, 0.0, 2.0, 2.0, snx, sny)
    d = GridSpec(0.0, 1.0 * ry, 2.0 * rx, 2.0 * ry, int(snx / rx), 1099)
    z = dem_on_grid(g, seed=5).astype(np.float32)
    z[np.random.default_rng(sny).random(z.shape) < 0.002] = np.nan
    dst = torch.full((d.ny, d.nx), -7.0, dtype=torch.float32, device="cuda")
    ag.auv_resample_kriging(torch.from_numpy(z).cuda(), g, dst, d, 6.0)
    torch.cuda.synchronize()
    want = orc.kriging(orc.Grid(g.x0, g.y0, g.dx, g.dy, snx, sny), z.astype(np.float64),
                       orc.Grid(d.x0, d.y0, d.dx, d.dy, d.nx, d.ny), 6.0)
    got = dst.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = ~np.isnan(want)
    assert (np.abs(got[ok] - want[ok]) / np.abs(want[ok])).max() <= 1e-5
