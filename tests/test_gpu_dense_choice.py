"""GPU parity of the dense form on both sides of the rule that picks its search on
bins of at least the radius (lists or rings): caps 8, 9, 16 and 17, densities just
below and above the limits of small grids (20 and 32 soundings per disk) and of
grids of 4096 tiles (40), against the FP64 oracle: counts, NaN masks and nearest
picks exact, depths within 1e-5 relative (FP32 sums of at most 17 terms)."""
import math

import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,cap,pop", [
    (60, 8, 31.0), (60, 8, 33.0), (60, 9, 19.0), (60, 9, 21.0), (60, 16, 19.0), (60, 16, 21.0),
    (60, 17, 12.0), (511, 9, 30.0), (512, 9, 39.0), (512, 16, 41.0),
])
def test_both_searches(orc, side, cap, pop):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    dx, r = 2.0, 6.0
    n = int(pop * (side * dx + 2 * r) ** 2 / (math.pi * r * r))
    g = GridSpec(10.0, 20.0, dx, dx, side, side)
    rng = np.random.default_rng(n + cap)
    x = g.x0 + rng.uniform(-r, side * dx + r, n)
    y = g.y0 + rng.uniform(-r, side * dx + r, n)
    snap = np.arange(n) % 5 == 0                     # ties, some on nodes
    x[snap] = g.x0 + np.round(x[snap] - g.x0)
    y[snap] = g.y0 + np.round(y[snap] - g.y0)
    z = -3000.0 + 9.0 * np.sin(x / 13.0) + rng.normal(0.0, 1.0, n)
    grid = ag.auv_grid_create(g)
    bins = ag.auv_bin_points(grid, *(torch.from_numpy(a).cuda() for a in (x, y, z)), r)
    out = ag.grid_idw(grid, bins, min_pts=1, max_pts=cap, with_counts=True, with_nearest=True,
                      algo=ag.AUV_ALGO_DENSE)
    torch.cuda.synchronize()
    oz, oc, on = orc.idw(orc.Grid(g.x0, g.y0, dx, dx, side, side), x, y, z, r, 2.0, 1, cap,
                         bin_log2=18)
    assert np.array_equal(out["cnt"].cpu().numpy(), oc)
    assert np.array_equal(out["nn_idx"].cpu().numpy(), on)
    gz = out["z"].cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(gz), np.isnan(oz))
    ok = ~np.isnan(oz)
    assert (np.abs(gz[ok] - oz[ok]) / np.abs(oz[ok])).max() <= 1e-5
