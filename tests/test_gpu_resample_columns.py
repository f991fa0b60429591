"""GPU parity of the column form of the bilinear and Catmull-Rom resamples against
the FP64 oracle where it can go wrong: sources of one and two nodes, destinations cut inside a
wave and inside a block's rows, ratios whose tap rows slide, repeat or jump,
source rectangles around and beyond the staged size, row lengths that are no
multiple of four, holes of NaN and infinities.

Bar (the definition's): NaN masks exact, values within 1e-5 relative."""
import numpy as np
import pytest
import torch

from gen import GridSpec, dem_on_grid

pytestmark = pytest.mark.gpu

REL = 1e-5


@pytest.mark.parametrize("method", ["bilinear", "bicubic"])
@pytest.mark.parametrize("snx,sny,dnx,dny,shift,hole", [
    (1, 1, 3, 5, 0.0, 0.0),
    (2, 300, 255, 33, 0.0, 0.0),
    (61, 47, 257, 31, 0.0, 0.02),
    (300, 201, 299, 200, 0.5, 0.01),     # infill
    (150, 130, 321, 251, -3.3, 0.02),    # beyond one end
    (700, 650, 301, 97, 0.0, 0.002),     # rows jump; rectangles halve the rows
    (3000, 40, 260, 39, 0.0, 0.001),     # beyond the staged size
    (500, 3, 1030, 7, 0.0, 0.01),
])
def test_resample_columns(orc, method, snx, sny, dnx, dny, shift, hole):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(10.0, -20.0, 2.0, 2.0, snx, sny)
    rx, ry = (1.0, 1.0) if shift == 0.5 else (snx / dnx, sny / dny)
    d = GridSpec(10.0, -20.0 + 2.0 * shift, 2.0 * rx, 2.0 * ry, dnx, dny)
    z = dem_on_grid(g, seed=7).astype(np.float32)
    u = np.random.default_rng(snx + dny).random(z.shape)
    z[u < hole] = np.nan
    z[u < hole / 4] = np.inf
    dst = torch.full((dny, dnx), -7.0, dtype=torch.float32, device="cuda")
    getattr(ag, f"auv_resample_{method}")(torch.from_numpy(z).cuda(), g, dst, d)
    torch.cuda.synchronize()
    want = getattr(orc, method)(orc.Grid(g.x0, g.y0, g.dx, g.dy, snx, sny),
                                z.astype(np.float64),
                                orc.Grid(d.x0, d.y0, d.dx, d.dy, dnx, dny))
    got = dst.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isfinite(got), np.isfinite(want))
    ok = np.isfinite(want)
    assert (np.abs(got[ok] - want[ok]) / np.abs(want[ok])).max() <= REL
