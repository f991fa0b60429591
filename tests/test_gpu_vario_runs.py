"""GPU parity of the semivariogram's run form against the oracle at the sizes
where it can go wrong: rows around the runs of 8 values, the 16 rows staged at
once and the 2048 values of a pass, lags around the groups of 8 and beyond the
grid, infinities beside NaN.  Bar: pair counts exact, values to 1e-9 relative
(FP64 sums of at most 1e6 positive terms in another order: n 2^-53)."""
import numpy as np
import pytest
import torch

from gen import GridSpec, dem_on_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nlags,hole", [
    (7, 1, 3, 0.0),
    (8, 9, 8, 0.2),
    (9, 257, 9, 0.0),
    (129, 8, 16, 0.1),
    (2047, 3, 17, 0.05),
    (2049, 17, 31, 0.05),
    (4100, 5, 1000, 0.02),
    (64, 1025, 33, 1.0),     # nothing but holes
])
def test_variogram_runs(orc, nx, ny, nlags, hole):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(0.0, 0.0, 2.0, 2.0, nx, ny)
    z = dem_on_grid(g, seed=3).astype(np.float32)
    u = np.random.default_rng(nx + ny).random(z.shape)
    z[u < hole] = np.nan
    z[u < hole / 3] = np.inf
    z[u < hole / 6] = -np.inf
    gx, gy, px, py = ag.auv_variogram(torch.from_numpy(z).cuda(), g, nlags)
    zo = np.where(np.isfinite(z), z, np.nan).astype(np.float64)
    ox, oy, opx, opy = orc.variogram(orc.Grid(0.0, 0.0, 2.0, 2.0, nx, ny), zo, nlags)
    assert np.array_equal(px, opx) and np.array_equal(py, opy)
    for a, b in ((gx, ox), (gy, oy)):
        assert np.allclose(a, b, rtol=1e-9, atol=0, equal_nan=True)
