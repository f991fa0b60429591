"""Resamples of grids whose origin is so far out that the coordinates of
neighbouring nodes coincide (2^55 m at 1 m and beyond): the nodes step by groups of
source cells, so a block's source rectangle may be larger than the spacings' ratio
says (258 columns instead of 155 at 2^58 m and a ratio of 0.6).
NaN masks exact, values within 1e-5 relative of the FP64 oracle, which maps the
axes with the same operations."""
import numpy as np
import pytest
import torch

from gen import GridSpec

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["bilinear", "bicubic", "kriging"])
@pytest.mark.parametrize("x0,y0", [(2.0 ** 55, 0.0), (2.0 ** 58, 0.0), (0.0, -2.0 ** 58),
                                   (2.0 ** 58, 2.0 ** 57), (4.5e6, -6.1e6)])
@pytest.mark.parametrize("rx,ry", [(1.0, 1.0), (0.6, 0.5), (0.6, 0.6)])
def test_far_origin(orc, method, x0, y0, rx, ry):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2505_22675_amd as ag
    nx, ny = 1500, 150
    s = GridSpec(x0, y0, 1.0, 1.0, nx, ny)
    d = GridSpec(x0, y0, rx, ry, int(nx / rx), int(ny / ry))
    rng = np.random.default_rng(3)
    z = (-500.0 + rng.normal(0.0, 2.0, (ny, nx))).astype(np.float32)
    z[rng.random(z.shape) < 0.001] = np.nan
    dst = torch.full((d.ny, d.nx), -7.0, dtype=torch.float32, device="cuda")
    extra = (3.0,) if method == "kriging" else ()
    getattr(ag, f"auv_resample_{method}")(torch.from_numpy(z).cuda(), s, dst, d, *extra)
    torch.cuda.synchronize()
    want = getattr(orc, method)(orc.Grid(s.x0, s.y0, s.dx, s.dy, nx, ny), z.astype(np.float64),
                                orc.Grid(d.x0, d.y0, d.dx, d.dy, d.nx, d.ny), *extra)
    got = dst.cpu().numpy().astype(np.float64)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    ok = ~np.isnan(want)
    assert (np.abs(got[ok] - want[ok]) / np.abs(want[ok])).max() <= 1e-5
