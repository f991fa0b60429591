"""GPU parity of batch items that the linear gather form does not take: caps
above 64 (window form), spacings whose offsets pass 2^24 lattice units, lattices
that are not linear and the largest radius (general gather form), beside ordinary
items, integer and general powers, tiles cut by the grid's edge.  The batch is
launched twice (the second replays its graph).  Against the FP64 oracle: counts,
NaN masks and nearest picks exact, depths within 1e-5 relative."""
import math

import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu

# soundings, columns, rows, spacing, radius, cap, power
ITEMS = {
    "caps": [(6000, 50, 33, 2.0, 6.0, 65, 2.0), (20000, 64, 17, 2.0, 6.0, 100, 1.0),
             (3000, 31, 48, 2.0, 6.0, 300, 3.0), (3000, 16, 16, 2.0, 6.0, 16, 2.0)],
    "caps, general power": [(6000, 50, 33, 2.0, 6.0, 65, 2.5), (9000, 30, 33, 2.0, 6.0, 80, 2.0)],
    "spacings": [(3000, 40, 33, 40.0, 30.0, 0, 2.0), (3000, 33, 50, 40.0, 60.0, 16, 3.0),
                 (4000, 45, 39, 3.3, 10.0, 0, 1.0), (4000, 45, 39, 3.3, 10.0, 64, 2.5),
                 (900, 9, 7, 300.0, 256.0, 4, 2.0), (3000, 40, 33, 2.0, 6.0, 0, 2.0)],
    "not batched": [(4000, 45, 39, 3.3, 10.0, 90, 2.0), (2000, 40, 40, 1.0, 6.0, 70, 2.0),
                    (3000, 40, 33, 2.0, 6.0, 100, 2.0)],
}


@pytest.mark.parametrize("name", list(ITEMS))
def test_items(orc, name):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    rng = np.random.default_rng(11)
    cases, items = [], []
    for k, (n, nx, ny, dx, r, cap, power) in enumerate(ITEMS[name]):
        g = GridSpec(1000.0 * k, -70.0, dx, dx, nx, ny)
        x = g.x0 + rng.uniform(-r, nx * dx + r, n)
        y = g.y0 + rng.uniform(-r, ny * dx + r, n)
        snap = np.arange(n) % 5 == 0                 # ties, some on nodes
        x[snap] = g.x0 + np.round((x[snap] - g.x0) * 2.0 / dx) * dx / 2.0
        y[snap] = g.y0 + np.round((y[snap] - g.y0) * 2.0 / dx) * dx / 2.0
        z = -1200.0 + rng.normal(0.0, 2.0, n)
        dev = [torch.from_numpy(a).cuda() for a in (x, y, z)]
        out = [torch.full((ny, nx), -3, dtype=t, device="cuda")
               for t in (torch.float32, torch.int32, torch.int32, torch.float32)]
        prm = ag.idw_params(power=power, radius=r, min_pts=2, max_pts=cap, algo=ag.AUV_ALGO_SPARSE)
        items.append(ag.batch_item(ag.make_desc(g.x0, g.y0, dx, dx, nx, ny), *dev, prm, *out))
        cases.append((g, x, y, z, r, power, cap, out, dev))
    batch = ag.Batch(items)
    for _ in range(2):
        for c in cases:
            for t in c[7]:
                t.fill_(-3)
        batch.launch()
        torch.cuda.synchronize()
        for g, x, y, z, r, power, cap, (zo, co, no, nz), _ in cases:
            oz, oc, on = orc.idw(orc.Grid(g.x0, g.y0, g.dx, g.dy, g.nx, g.ny), x, y, z, r, power, 2,
                                 cap, bin_log2=max(12, math.ceil(math.log2(r * 65536))))
            assert np.array_equal(co.cpu().numpy(), oc)
            assert np.array_equal(no.cpu().numpy(), on)
            assert np.array_equal(nz.cpu().numpy()[on >= 0], z[on[on >= 0]].astype(np.float32))
            gz = zo.cpu().numpy().astype(np.float64)
            assert np.array_equal(np.isnan(gz), np.isnan(oz))
            ok = ~np.isnan(oz)
            assert (np.abs(gz[ok] - oz[ok]) / np.abs(oz[ok])).max() <= 1e-5
    batch.close()
