"""Membership at the largest radius (256 m, 2^24 lattice units): a sounding on a
node's row or column at exactly the radius belongs to the node, one lattice unit
(2^-16 m) further does not.  2^24 + 1 is no FP32 number, so an offset rounded to
FP32 cannot tell the two apart.  Against the FP64 oracle: counts, NaN masks and
nearest picks exact, depths within 1e-5 relative (sums of at most 32 terms)."""
import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu

UNIT = 2.0 ** -16


def _soundings(g, r, extra):
    """Around every node: soundings at r + k units, k in -1..2, along both axes
    and diagonally, plus `extra` at random."""
    xs = g.x0 + (np.arange(g.nx) + 0.5) * g.dx
    ys = g.y0 + (np.arange(g.ny) + 0.5) * g.dy
    x, y = [], []
    for b in xs:
        for a in ys:
            for k in range(-1, 3):
                d = r + k * UNIT
                for sx, sy in ((1, 0), (-1, 0), (0, 1), (0, -1)):
                    x.append(b + sx * d)
                    y.append(a + sy * d)
            x.append(b + r * 0.6)
            y.append(a + r * 0.8)
    rng = np.random.default_rng(extra)
    x = np.concatenate([x, rng.uniform(xs[0] - r, xs[-1] + r, extra)])
    y = np.concatenate([y, rng.uniform(ys[0] - r, ys[-1] + r, extra)])
    return x, y, -900.0 + rng.normal(0.0, 5.0, x.size)


@pytest.mark.parametrize("algo,cap", [("SPARSE", 0), ("SPARSE", 3), ("DENSE", 5), ("DENSE", 16)])
@pytest.mark.parametrize("dx", [300.0, 700.0])   # overlapping disks, apart
@pytest.mark.parametrize("r", [256.0, 256.0 - UNIT])
def test_members_at_the_radius(orc, r, dx, algo, cap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(64.0, -32.0, dx, dx, 9, 5)
    x, y, z = _soundings(g, r, 40)
    grid = ag.auv_grid_create(g)
    bins = ag.auv_bin_points(grid, *(torch.from_numpy(a).cuda() for a in (x, y, z)), r)
    out = ag.grid_idw(grid, bins, min_pts=1, max_pts=cap, with_counts=True, with_nearest=True,
                      algo=getattr(ag, "AUV_ALGO_" + algo))
    idx = torch.empty((g.ny, g.nx), dtype=torch.int32, device="cuda")
    ag.auv_interp_nearest(grid, bins, r, idx)
    torch.cuda.synchronize()
    oz, oc, on = orc.idw(orc.Grid(g.x0, g.y0, dx, dx, g.nx, g.ny), x, y, z, r, 2.0, 1, cap,
                         bin_log2=-1)
    assert np.array_equal(out["cnt"].cpu().numpy(), oc)
    assert np.array_equal(out["nn_idx"].cpu().numpy(), on)
    assert np.array_equal(idx.cpu().numpy(), on)
    gz = out["z"].cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(gz), np.isnan(oz))
    ok = ~np.isnan(oz)
    assert (np.abs(gz[ok] - oz[ok]) / np.abs(oz[ok])).max() <= 1e-5


@pytest.mark.parametrize("k", [0, 1])
def test_one_sounding_at_the_radius(orc, k):
    """The only sounding, at 2^24 + k units: the nearest pick and the value exist
    for k = 0 alone."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    g = GridSpec(0.0, 0.0, 300.0, 300.0, 3, 3)
    x = np.array([450.0 + 256.0 + k * UNIT])
    y = np.array([450.0])
    z = np.array([-700.0])
    grid = ag.auv_grid_create(g)
    bins = ag.auv_bin_points(grid, *(torch.from_numpy(a).cuda() for a in (x, y, z)), 256.0)
    out = ag.grid_idw(grid, bins, min_pts=1, max_pts=0, with_counts=True, with_nearest=True)
    idx = torch.empty((3, 3), dtype=torch.int32, device="cuda")
    ag.auv_interp_nearest(grid, bins, 256.0, idx)
    torch.cuda.synchronize()
    for a in (out["nn_idx"], idx):
        assert a[1, 1].item() == (0 if k == 0 else -1)
    assert out["cnt"][1, 1].item() == 1 - k
    assert torch.isnan(out["z"][1, 1]).item() == (k == 1)
