"""GPU parity of dense batch items around the densities where their search
changes, each against the FP64 oracle.  Items of cap 16 without a table: up to 3
caps (48 soundings) per disk of 6 m the default 8 m bins and the form by lists,
above it the ring search on bins halved until they hold a few soundings: 4 m up
to 103 per disk, 2 m up to 414, then 1 m.  Caps under 8 count as 8.  The batch is
launched twice.  Bar: counts, NaN masks and nearest picks exact, depths within
1e-5 relative (FP32 sums of at most 16 terms)."""
import math

import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu

R, DX, SIDE = 6.0, 2.0, 40


@pytest.mark.parametrize("cap,pops", [
    (16, (46.0, 50.0, 101.0, 107.0, 408.0, 420.0)),
    (4, (23.0, 25.0, 50.0, 54.0)),
])
def test_each_side_of_a_halving(orc, cap, pops):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    rng = np.random.default_rng(cap)
    cases, items = [], []
    for k, pop in enumerate(pops):
        n = round(pop * (SIDE * DX + 2 * R) ** 2 / (math.pi * R * R))
        g = GridSpec(500.0 * k, 30.0, DX, DX, SIDE, SIDE)
        x = g.x0 + rng.uniform(-R, SIDE * DX + R, n)
        y = g.y0 + rng.uniform(-R, SIDE * DX + R, n)
        snap = np.arange(n) % 7 == 0                 # ties, some on nodes
        x[snap] = g.x0 + np.round(x[snap] - g.x0)
        y[snap] = g.y0 + np.round(y[snap] - g.y0)
        z = -2200.0 + rng.normal(0.0, 2.0, n)
        dev = [torch.from_numpy(a).cuda() for a in (x, y, z)]
        out = [torch.full((SIDE, SIDE), -3, dtype=t, device="cuda")
               for t in (torch.float32, torch.int32, torch.int32)]
        items.append(ag.batch_item(ag.make_desc(g.x0, g.y0, DX, DX, SIDE, SIDE), *dev,
                                   ag.idw_params(radius=R, min_pts=1, max_pts=cap), *out))
        cases.append((g, x, y, z, out, dev))
    batch = ag.Batch(items)
    for _ in range(2):
        for c in cases:
            for t in c[4]:
                t.fill_(-3)
        batch.launch()
        torch.cuda.synchronize()
        for g, x, y, z, (zo, co, no), _ in cases:
            oz, oc, on = orc.idw(orc.Grid(g.x0, g.y0, DX, DX, SIDE, SIDE), x, y, z, R, 2.0, 1, cap,
                                 bin_log2=18)
            assert np.array_equal(co.cpu().numpy(), oc)
            assert np.array_equal(no.cpu().numpy(), on)
            gz = zo.cpu().numpy().astype(np.float64)
            assert np.array_equal(np.isnan(gz), np.isnan(oz))
            ok = ~np.isnan(oz)
            assert (np.abs(gz[ok] - oz[ok]) / np.abs(oz[ok])).max() <= 1e-5
    batch.close()
