"""GPU parity of the dense form on subdivided bins (batch items that no tuning
table sets) against the FP64 oracle: populations around the step where the
subdivision starts and far above it, soundings gathered in a corner (most nodes
reach nothing, so the search's annuli double), caps of 1 to 16.

Bar (the definition's): counts, NaN masks and nearest picks exact; depths
within 1e-5 relative (FP32 sums of at most 16 terms relative to a member's
depth)."""
import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu

REL = 1e-5


@pytest.mark.parametrize("n,nx,ny,r,cap,corner", [
    (700, 40, 33, 6.0, 16, 1.0),        # about 16 per disk: bins as planned
    (1500, 40, 33, 6.0, 16, 1.0),       # first subdivision
    (30000, 33, 47, 6.0, 16, 1.0),
    (30000, 64, 64, 6.0, 5, 0.3),       # nine tenths of the grid out of reach
    (60000, 17, 9, 20.0, 1, 0.6),       # reach of ten nodes, hundreds of bins per side
    (20000, 130, 5, 3.3, 9, 0.5),
])
def test_dense_subdivided_bins(orc, n, nx, ny, r, cap, corner):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(100.0, -300.0, 2.0, 2.0, nx, ny)
    rng = np.random.default_rng(n + nx)
    x = g.x0 + rng.uniform(-r, corner * nx * 2.0, n)
    y = g.y0 + rng.uniform(-r, corner * ny * 2.0, n)
    snap = np.arange(n) % 3 == 0                     # lattice ties, hits on nodes
    x[snap] = g.x0 + np.round(x[snap] - g.x0)
    y[snap] = g.y0 + np.round(y[snap] - g.y0)
    z = -4000.0 + 30.0 * np.sin(x / 17.0) + rng.normal(0, 2.0, n)
    dev = [torch.from_numpy(a).cuda() for a in (x, y, z)]
    zo = torch.full((ny, nx), -1.0, dtype=torch.float32, device="cuda")
    co = torch.full((ny, nx), -7, dtype=torch.int32, device="cuda")
    no = torch.full((ny, nx), -7, dtype=torch.int32, device="cuda")
    prm = ag.idw_params(power=2.0, radius=r, min_pts=1, max_pts=cap)
    b = ag.Batch([ag.batch_item(ag.make_desc(g.x0, g.y0, 2.0, 2.0, nx, ny), *dev, prm, zo, co,
                                no)])
    assert b.item_plan(0)[1] == ag.AUV_ALGO_DENSE
    for _ in range(2):
        b.launch()
    torch.cuda.synchronize()
    oz, oc, on = orc.idw(orc.Grid(g.x0, g.y0, 2.0, 2.0, nx, ny), x, y, z, r, 2.0, 1, cap,
                         bin_log2=16)
    assert np.array_equal(co.cpu().numpy(), oc)
    assert np.array_equal(no.cpu().numpy(), on)
    gz = zo.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(gz), np.isnan(oz))
    ok = ~np.isnan(oz)
    assert (np.abs(gz[ok] - oz[ok]) / np.abs(oz[ok])).max() <= REL
    b.close()
