"""GPU parity of the gather form (one lane per node, quarter-tile lists; the
sparse form of auv_interp_idw and auv_interp_nearest) against the FP64 oracle,
at the sizes where it can go wrong: tiles cut by the grid's edge, batches of
exactly and just over 64 candidates, more than 64 bin rows per tile, caps
around the rounds of its register list (8), ties and coincident soundings,
node lattices that are not linear, offsets beyond the FP32 integers.

Bar (the definition's): counts, NaN masks and nearest picks exact; depths
within 1e-5 relative (FP32 weights and sums of at most a few hundred terms
relative to a member's depth: about n 2^-24 of the members' depth range, far
below 1e-5 of the depth itself)."""
import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu

REL = 1e-5


@pytest.fixture(scope="module")
def ag():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    ag.load_library()
    return ag


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _check(ag, orc, g, x, y, z, r, power, min_pts, kcap, bin_log2=0, orc_log2=-1):
    grid = ag.auv_grid_create(g)
    bins = ag.auv_bin_points(grid, _dev(x), _dev(y), _dev(z), r, bin_log2)
    out = ag.grid_idw(grid, bins, power=power, min_pts=min_pts, max_pts=kcap,
                      with_counts=True, with_nearest=True, algo=ag.AUV_ALGO_SPARSE)
    plain = ag.grid_idw(grid, bins, power=power, min_pts=min_pts, max_pts=kcap,
                        algo=ag.AUV_ALGO_SPARSE)
    idx = torch.empty((g.ny, g.nx), dtype=torch.int32, device="cuda")
    nz = torch.empty((g.ny, g.nx), dtype=torch.float32, device="cuda")
    ag.auv_interp_nearest(grid, bins, r, idx, nz)
    torch.cuda.synchronize()
    og = orc.Grid(g.x0, g.y0, g.dx, g.dy, g.nx, g.ny)
    oz, oc, on = orc.idw(og, x, y, z, r, power, min_pts, kcap, bin_log2=orc_log2)
    for res in (out["z"], plain["z"]):
        gz = res.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isnan(gz), np.isnan(oz))
        ok = ~np.isnan(oz)
        assert not ok.any() or (np.abs(gz[ok] - oz[ok]) / np.abs(oz[ok])).max() <= REL
    assert np.array_equal(out["cnt"].cpu().numpy(), oc)
    for i, n in ((out["nn_idx"], out["nn_z"]), (idx, nz)):
        assert np.array_equal(i.cpu().numpy(), on)
        have = on >= 0
        assert np.array_equal(n.cpu().numpy()[have], z[on[have]].astype(np.float32))
        assert np.isnan(n.cpu().numpy()[~have]).all()
    lo, hi = orc.idw_bounds(og, x, y, z, r, kcap, bin_log2=orc_log2)
    gz = out["z"].cpu().numpy()
    ok = ~np.isnan(gz)
    assert (gz[ok] >= lo[ok].astype(np.float32)).all() and (gz[ok] <= hi[ok].astype(np.float32)).all()
    return oc


def _field(seed, n, g, r):
    rng = np.random.default_rng(seed)
    x = g.x0 + rng.uniform(-r, g.nx * g.dx + r, n)
    y = g.y0 + rng.uniform(-r, g.ny * g.dy + r, n)
    return x, y, -4000.0 - 50.0 * np.sin(x / 37.0) + rng.normal(0, 2.0, n)


@pytest.mark.parametrize("nx,ny,dx,r,n,kcap,power", [
    (1, 1, 2.0, 6.0, 64, 0, 2.0),            # one node, one batch at most
    (1, 1, 2.0, 6.0, 65, 7, 1.0),
    (7, 9, 2.0, 6.0, 40, 8, 2.0),            # cut tiles, the second column of quarters missing
    (8, 8, 0.5, 1.25, 300, 9, 3.0),          # a whole tile, a cap of one round and one more
    (12, 4, 1.0, 3.0, 500, 16, 2.5),         # general power, no second row of quarters
    (65, 33, 3.3, 10.0, 4000, 0, 2.0),       # lattice not linear
    (33, 21, 1000.0 / 255.0, 9.0, 6000, 33, 2.0),  # not linear, more rounds than the dense form keeps
    (20, 13, 40.0, 230.0, 900, 40, 2.0),     # offsets beyond 2^24, long radius
    (20, 13, 40.0, 230.0, 900, 0, 2.5),
])
def test_gather_sizes(ag, orc, nx, ny, dx, r, n, kcap, power):
    g = GridSpec(-250.0, 1234.5, dx, dx, nx, ny)
    x, y, z = _field(nx * 31 + ny, n, g, r)
    x[::29], z[5::41] = np.nan, np.inf
    _check(ag, orc, g, x, y, z, r, power, 2, kcap)


@pytest.mark.parametrize("kcap,snap", [(0, 0.5), (3, 0.25), (8, 0.5), (20, 0.125)])
def test_gather_ties_and_hits(ag, orc, kcap, snap):
    """Soundings snapped to the node lattice: equal distances at the cap and at
    the radius, several soundings on one node."""
    g = GridSpec(-3.0, 5.0, 0.5, 0.5, 37, 29)
    x, y, z = _field(91 + kcap, 4000, g, 1.0)
    x = g.x0 + np.round((x - g.x0) / snap) * snap
    y = g.y0 + np.round((y - g.y0) / snap) * snap
    x[:400] = g.x0 + (np.arange(400) % 37 + 0.5) * 0.5
    y[:400] = g.y0 + (np.arange(400) // 37 + 0.5) * 0.5
    oc = _check(ag, orc, g, x, y, z, 1.0, 2.0, 3, kcap)
    assert kcap == 0 or (oc == kcap).sum() > 100


def test_gather_many_bin_rows(ag, orc):
    """Bins of 1/16 m: a tile's candidates lie in more than 64 bin rows."""
    g = GridSpec(0.0, 0.0, 1.0, 1.0, 30, 26)
    x, y, z = _field(7, 2500, g, 2.0)
    _check(ag, orc, g, x, y, z, 2.0, 2.0, 1, 5, bin_log2=12)
