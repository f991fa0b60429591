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


@pytest.mark.parametrize("tile", [(16, 4), (4, 16), (64, 1)])
def test_dense_tiles_of_narrow_items(orc, tmp_path, tile):
    """Items one node wide or high whose planned tile has more units than 8 x 8
    tiles would: the work list has room for them."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    rng = np.random.default_rng(5)
    items, data = [], []
    for k in range(60):
        nx, ny = (1, 9) if k % 2 else (9, 1)
        x, y = rng.uniform(-6, nx * 2.0 + 6, 300), rng.uniform(-6, ny * 2.0 + 6, 300)
        z = -300.0 + rng.normal(0, 2.0, 300)
        dev = [torch.from_numpy(a).cuda() for a in (x, y, z)]
        zo = torch.full((ny, nx), -1.0, dtype=torch.float32, device="cuda")
        prm = ag.idw_params(power=2.0, radius=6.0, min_pts=1, max_pts=16)
        items.append(ag.batch_item(ag.make_desc(0.0, 0.0, 2.0, 2.0, nx, ny), *dev, prm, zo, None,
                                   None))
        data.append((nx, ny, x, y, z, zo, dev))
    pop = 300 / ((1 * 2.0 + 12.0) * (9 * 2.0 + 12.0)) * np.pi * 36.0
    table = tmp_path / "tune.txt"
    table.write_text(f"class {int(np.floor(np.log2(pop + 1)))} {round(np.log2(9))} bin_log2 17 "
                     f"algo {ag.AUV_ALGO_DENSE} tile {tile[0]} {tile[1]} ms 1\n")
    b = ag.Batch(items, str(table))
    assert all(b.item_plan_full(i) == (17, ag.AUV_ALGO_DENSE, *tile) for i in range(60))
    b.launch()
    torch.cuda.synchronize()
    for nx, ny, x, y, z, zo, _ in data:
        oz, _, _ = orc.idw(orc.Grid(0.0, 0.0, 2.0, 2.0, nx, ny), x, y, z, 6.0, 2.0, 1, 16,
                           bin_log2=-1)
        gz = zo.cpu().numpy().astype(np.float64)
        assert (np.abs(gz - oz) / np.abs(oz)).max() <= REL
    b.close()
