"""Calls of 2^32 nodes and more: more node tiles than one launch takes (HIP
launches fewer than 2^32 threads), as a single grid and as the items of a
batch; and rows so long that seven of them pass 32-bit byte offsets.  A few
soundings at each grid's corners and centre; every node within reach of one is
checked against 64-bit arithmetic, and no other has a value."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DX = 0.25


def _ready():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.mem_get_info()[0] < 28 << 30:
        pytest.skip("needs 28 GB of GPU memory")
    import paper_2505_22675_amd as ag
    return ag


def _soundings(nx, ny):
    w, h = nx * DX, ny * DX
    at = [(0.3, 0.4), (w - 0.3, 0.2), (0.1, h - 0.2), (w - 0.3, h - 0.4), (w / 2, h / 2),
          (w - 0.35, h - 0.3)]
    x, y = (np.array(v) for v in zip(*at))
    return x, y, -np.arange(10.0, 10.0 + x.size)


def _check(z, nx, ny, r):
    x, y, d = _soundings(nx, ny)
    R2 = np.rint(r * 65536) ** 2
    want = {}
    for xs, ys in zip(x, y):
        for a in range(max(0, int((ys - r) / DX) - 1), min(ny, int((ys + r) / DX) + 2)):
            for b in range(max(0, int((xs - r) / DX) - 1), min(nx, int((xs + r) / DX) + 2)):
                ex = np.rint(x * 65536) - (b + 0.5) * DX * 65536
                ey = np.rint(y * 65536) - (a + 0.5) * DX * 65536
                m = ex * ex + ey * ey <= R2
                if m.any():
                    q = ((x - (b + 0.5) * DX) ** 2 + (y - (a + 0.5) * DX) ** 2)[m]
                    hit = (ex * ex + ey * ey)[m] == 0   # a hit's depth stands alone
                    w = hit.astype(float) if hit.any() else 1.0 / q
                    want[a, b] = (w * d[m]).sum() / w.sum()
    have = sum(int(torch.isfinite(z[i:i + 4096]).sum().item()) for i in range(0, ny, 4096))
    assert have == len(want)
    k = torch.tensor(list(want), dtype=torch.int64, device="cuda")
    got = z[k[:, 0], k[:, 1]].double().cpu().numpy()
    ref = np.array(list(want.values()))
    assert (np.abs(got - ref) / np.abs(ref)).max() <= 1e-5


@pytest.mark.parametrize("algo,cap", [("SPARSE", 0), ("DENSE", 4)])
def test_call(algo, cap):
    ag = _ready()
    n, r = 65535, 0.75
    grid = ag.auv_grid_create(ag.make_desc(0.0, 0.0, DX, DX, n, n))
    bins = ag.auv_bin_points(grid, *(torch.from_numpy(a).cuda() for a in _soundings(n, n)), r, 20)
    z = torch.empty((n, n), dtype=torch.float32, device="cuda")
    prm = ag.idw_params(radius=r, min_pts=1, max_pts=cap, algo=getattr(ag, "AUV_ALGO_" + algo))
    ag.auv_interp_idw(grid, bins, prm, z)
    torch.cuda.synchronize()
    _check(z, n, n, r)


@pytest.mark.parametrize("cap", [0, 4])
def test_batch(cap):
    ag = _ready()
    nx, ny, r = 65504, 32800, 1.9
    algo = ag.AUV_ALGO_DENSE if cap else ag.AUV_ALGO_SPARSE
    keep, items = [], []
    for _ in range(2):
        p = [torch.from_numpy(a).cuda() for a in _soundings(nx, ny)]
        z = torch.empty((ny, nx), dtype=torch.float32, device="cuda")
        keep.append((p, z))
        items.append(ag.batch_item(ag.make_desc(0.0, 0.0, DX, DX, nx, ny), *p,
                                   ag.idw_params(radius=r, min_pts=1, max_pts=cap, algo=algo),
                                   z.view(-1)))
    batch = ag.Batch(items)
    batch.launch()
    torch.cuda.synchronize()
    batch.close()
    for _, z in keep:
        _check(z, nx, ny, r)


@pytest.mark.parametrize("nx,dx,cap", [
    (160_000_000, 1e-4, 0),            # 6.55 lattice units: not linear
    (130_000_000, 2.0 ** -13, 0),      # linear
    (130_000_000, 2.0 ** -13, 70),     # beyond the gather form's caps
])
def test_long_rows(nx, dx, cap):
    """One sounding by the row's end in the first, seventh, eighth and last row."""
    ag = _ready()
    ny, dy, r = 9, 1.0, 0.01
    end = nx * dx
    rows = [0, 6, 7, 8]
    x = np.array([end - 1.0, end - 2.0, end - 0.01, end - 10.0])
    y = np.array([a + 0.5 + 0.002 for a in rows])
    d = -np.arange(20.0, 24.0)
    grid = ag.auv_grid_create(ag.make_desc(0.0, 0.0, dx, dy, nx, ny))
    bins = ag.auv_bin_points(grid, *(torch.from_numpy(a).cuda() for a in (x, y, d)), r, 20)
    z = torch.empty((ny, nx), dtype=torch.float32, device="cuda")
    prm = ag.idw_params(radius=r, min_pts=1, max_pts=cap, algo=ag.AUV_ALGO_SPARSE)
    ag.auv_interp_idw(grid, bins, prm, z)
    torch.cuda.synchronize()
    have = 0
    for xs, ys, a, depth in zip(x, y, rows, d):
        b = np.arange(max(0, int((xs - r) / dx) - 3), min(nx, int((xs + r) / dx) + 4))
        ex = np.rint(xs * 65536) - np.rint(((b + 0.5) * dx) * 65536)
        ey = np.rint(ys * 65536) - np.rint((a + 0.5) * dy * 65536)
        member = ex * ex + ey * ey <= np.rint(r * 65536) ** 2
        got = z[a, int(b[0]):int(b[-1]) + 1].cpu().numpy()
        assert np.array_equal(np.isfinite(got), member)
        assert (got[member] == np.float32(depth)).all()
        have += int(member.sum())
    assert have == sum(int(torch.isfinite(row).sum().item()) for row in z)
