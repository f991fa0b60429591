"""GPU parity of the dense form on bins of at least the radius (the gather form's
lists, one pass, sorted register lists of 8, 16 and 32) against the FP64 oracle:
caps at the list lengths, tiles cut by the grid's edge, more candidates than a
batch, few members, ties and coincident soundings, node lattices that are not
linear, offsets beyond 2^24, bins just at and just below the radius.

Bar (the definition's): counts, NaN masks and nearest picks exact; depths
within 1e-5 relative (FP32 sums of at most 32 terms relative to a member's
depth)."""
import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu

REL = 1e-5


@pytest.mark.parametrize("n,nx,ny,dx,r,cap,min_pts,power,bin_log2", [
    (9000, 64, 40, 2.0, 6.0, 16, 1, 2.0, 0),
    (9000, 65, 41, 2.0, 6.0, 8, 3, 1.0, 0),
    (5000, 33, 47, 2.0, 6.0, 9, 0, 3.0, 0),
    (20000, 50, 31, 2.0, 6.0, 32, 1, 2.5, 0),
    (300, 31, 29, 2.0, 6.0, 17, 2, 2.0, 0),
    (4000, 40, 40, 3.3, 10.0, 16, 1, 2.0, 0),     # lattice not linear
    (3000, 9, 7, 60.0, 120.0, 1, 1, 2.0, 0),      # offsets above 2^24
    (9000, 40, 40, 2.0, 4.0, 16, 1, 2.0, 18),     # bins of exactly the radius
    (9000, 40, 40, 2.0, 4.5, 16, 1, 2.0, 18),     # just below: ring search
])
def test_dense_by_lists(orc, n, nx, ny, dx, r, cap, min_pts, power, bin_log2):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(40.0, -70.0, dx, dx, nx, ny)
    rng = np.random.default_rng(n + cap)
    x = g.x0 + rng.uniform(-r, nx * dx + r, n)
    y = g.y0 + rng.uniform(-r, ny * dx + r, n)
    snap = np.arange(n) % 4 == 0                     # ties, some on nodes
    x[snap] = g.x0 + np.round((x[snap] - g.x0) * 2.0 / dx) * dx / 2.0
    y[snap] = g.y0 + np.round((y[snap] - g.y0) * 2.0 / dx) * dx / 2.0
    z = -2000.0 + 9.0 * np.sin(x / 13.0) + rng.normal(0, 1.0, n)
    grid = ag.auv_grid_create(g)
    bins = ag.auv_bin_points(grid, *(torch.from_numpy(a).cuda() for a in (x, y, z)), r, bin_log2)
    out = ag.grid_idw(grid, bins, power=power, min_pts=min_pts, max_pts=cap, with_counts=True,
                      with_nearest=True, algo=ag.AUV_ALGO_DENSE)
    torch.cuda.synchronize()
    oz, oc, on = orc.idw(orc.Grid(g.x0, g.y0, dx, dx, nx, ny), x, y, z, r, power, min_pts, cap,
                         bin_log2=-1)
    assert np.array_equal(out["cnt"].cpu().numpy(), oc)
    assert np.array_equal(out["nn_idx"].cpu().numpy(), on)
    gz = out["z"].cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(gz), np.isnan(oz))
    ok = ~np.isnan(oz)
    assert (np.abs(gz[ok] - oz[ok]) / np.abs(oz[ok])).max() <= REL
