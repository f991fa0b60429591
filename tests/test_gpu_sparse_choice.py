"""GPU parity of the sparse calls at the edges of the rule that picks their form
(gather or window), against the FP64 oracle: about 64 bin rows per node tile and
far more (radii of a few percent of the spacing), grids of 2M nodes around four
soundings expected per tile, with and without a cap, empty bin rows, and node
lattices that only the gather form takes.  Counts, NaN masks and nearest picks
exact, depths within 1e-5 relative (FP32 sums of at most a few dozen terms)."""
import math

import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nx,ny,dx,r,cap,bin_log2", [
    (4000, 41, 30, 16.0, 2.0, 0, 17),       # 60 bin rows per tile
    (4000, 41, 30, 16.0, 1.9, 0, 16),       # 116
    (4000, 41, 30, 16.0, 0.3, 0, 0),        # 226
    (4000, 41, 30, 16.0, 0.3, 4, 0),        # the same with a cap
    (4000, 41, 30, 16.3, 0.3, 0, 0),        # the same on a lattice that is not linear
    (300, 41, 30, 16.0, 3.0, 0, 0),         # mostly empty bin rows
    (21000, 1500, 1400, 2.0, 4.5, 0, 0),    # two expected per tile
    (45000, 1500, 1400, 2.0, 4.5, 0, 0),    # four
    (45000, 1500, 1400, 2.0, 4.5, 16, 0),
    (45000, 1500, 1390, 2.0, 4.5, 0, 0),    # just under 32768 tiles
])
def test_sparse_forms(orc, n, nx, ny, dx, r, cap, bin_log2):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(100.0, -300.0, dx, dx, nx, ny)
    rng = np.random.default_rng(n + nx)
    x = g.x0 + rng.uniform(-r, nx * dx + r, n)
    y = g.y0 + rng.uniform(-r, ny * dx + r, n)
    near = np.arange(n) % 3 == 0                    # within reach of a node, some on it
    m = int(near.sum())
    x[near] = g.x0 + (rng.integers(0, nx, m) + 0.5) * dx + rng.uniform(-r, r, m) * (np.arange(m) % 4 > 0)
    y[near] = g.y0 + (rng.integers(0, ny, m) + 0.5) * dx + rng.uniform(-r, r, m) * (np.arange(m) % 4 > 0)
    z = -1500.0 + rng.normal(0.0, 3.0, n)
    grid = ag.auv_grid_create(g)
    bins = ag.auv_bin_points(grid, *(torch.from_numpy(a).cuda() for a in (x, y, z)), r, bin_log2)
    out = ag.grid_idw(grid, bins, min_pts=1, max_pts=cap, with_counts=True, with_nearest=True)
    plain = ag.grid_idw(grid, bins, min_pts=1, max_pts=cap)
    idx = torch.empty((ny, nx), dtype=torch.int32, device="cuda")
    ag.auv_interp_nearest(grid, bins, r, idx)
    torch.cuda.synchronize()
    oz, oc, on = orc.idw(orc.Grid(g.x0, g.y0, dx, dx, nx, ny), x, y, z, r, 2.0, 1, cap,
                         bin_log2=max(12, math.ceil(math.log2(r * 65536))))
    assert np.array_equal(out["cnt"].cpu().numpy(), oc)
    assert np.array_equal(out["nn_idx"].cpu().numpy(), on)
    assert np.array_equal(idx.cpu().numpy(), on)
    for res in (out["z"], plain["z"]):
        gz = res.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isnan(gz), np.isnan(oz))
        ok = ~np.isnan(oz)
        assert (np.abs(gz[ok] - oz[ok]) / np.abs(oz[ok])).max() <= 1e-5
