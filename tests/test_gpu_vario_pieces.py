"""GPU parity of the semivariogram against the oracle on short wide grids, whose
bands of rows are split into pieces of columns: around the 64 columns that a
piece has at least, rows around the bands of eight, lags longer than a piece.
Bar: pair counts exact, values to 1e-9 relative (FP64 sums of at most 1e6
positive terms in another order: n 2^-53)."""
import numpy as np
import pytest
import torch

from gen import GridSpec, dem_on_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nlags,hole", [
    (127, 8, 9, 0.1),
    (128, 8, 9, 0.1),
    (300, 20, 10, 0.1),
    (1537, 7, 70, 0.0),
    (5003, 8, 600, 0.02),
    (20011, 17, 33, 0.05),
    (4099, 100, 1, 0.3),
])
def test_variogram_pieces(orc, nx, ny, nlags, hole):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(0.0, 0.0, 0.5, 0.5, nx, ny)
    z = dem_on_grid(g, seed=3).astype(np.float32)
    z[np.random.default_rng(nx + ny).random(z.shape) < hole] = np.nan
    gx, gy, px, py = ag.auv_variogram(torch.from_numpy(z).cuda(), g, nlags)
    ox, oy, opx, opy = orc.variogram(orc.Grid(0.0, 0.0, 0.5, 0.5, nx, ny), z.astype(np.float64),
                                     nlags)
    assert np.array_equal(px, opx) and np.array_equal(py, opy)
    for a, b in ((gx, ox), (gy, oy)):
        assert np.allclose(a, b, rtol=1e-9, atol=0, equal_nan=True)
