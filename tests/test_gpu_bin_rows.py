"""GPU parity of the row binning against the oracle, exact, at the sizes where
its forms meet: rows around the 1024, 2048 and 3072 keys that a sort block
holds and the 8192 above it, bins around 64 members, soundings around the call
size from which the histogram takes larger blocks, few and many bin rows, in
ping order and in none, some invalid or outside."""
import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nx,ny,d,r,ordered", [
    (1, 3, 3, 1.0, 1.0, False),
    (4095, 60, 10, 2.0, 6.0, False),        # 4 rows of about 1000 keys
    (9000, 400, 14, 2.0, 6.0, False),       # 6 rows of about 1500, few per bin
    (21000, 900, 24, 2.0, 6.0, True),       # rows around 2048 and 3072
    (65535, 1500, 60, 2.0, 6.0, False),
    (65537, 1500, 60, 2.0, 6.0, False),     # larger histogram blocks
    (120000, 2000, 30, 2.0, 6.0, True),     # rows of about 8192 and more
    (200000, 40, 300, 1.0, 2.0, False),     # bins over 64
    (90000, 64, 1400, 1.0, 2.0, True),      # 700 rows
])
def test_row_binning(orc, n, nx, ny, d, r, ordered):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(-50.0, 700.0, d, d, nx, ny)
    rng = np.random.default_rng(n)
    x = g.x0 + rng.uniform(-2 * r, nx * d + r, n)
    y = g.y0 + rng.uniform(-r, ny * d + 2 * r, n)
    if ordered:
        y.sort()
    z = -rng.uniform(100.0, 200.0, n)
    z[::97] = np.nan
    bins = ag.auv_bin_points(ag.auv_grid_create(g),
                             *(torch.from_numpy(a).cuda() for a in (x, y, z)), r, 0)
    cs, perm, counts = ag.auv_bins_export(bins)
    used = ag.auv_bins_info(bins)[3]
    ocs, operm, obad, oout = orc.bin_points(orc.Grid(g.x0, g.y0, d, d, nx, ny), x, y, z, r, used)
    assert counts == (operm.shape[0], obad, oout)
    assert np.array_equal(cs.cpu().numpy(), ocs)
    assert np.array_equal(perm.cpu().numpy(), operm)
