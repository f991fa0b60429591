"""Performance cases: the gridding work a program asks of this library, through
its public entry points, over the range of sizes and options it is used with.

    listed()            the standing cases
    draw(rng)           one more case from the same ranges
    prepare(case, seed) inputs and handles a program holds before the call
    run(state)          one pass through the entry points, returning its outputs
    work(case)          bytes and operations one pass cannot do without
    exact(case, seed)   the same outputs in 64 bits, in plain torch

Seven kinds of work:
    step       bin, IDW with the nearest pick, bilinear 2x: the mapping step
    grid       bin and IDW of scattered soundings
    nearest    bin and nearest-neighbour gridding
    batch      many uneven tiles planned once and launched as one batch
    serve      requests into resident vehicle grids, and the grids read out
    resample   bilinear, Catmull-Rom or kriging resample of a grid with holes
    variogram  the empirical semivariogram of a grid with holes
"""
import math
import random

import numpy as np
import torch

import paper_2505_22675_amd as ag

_LATTICE = 65536.0


# ------------------------------------------------------------------- cases --

def listed():
    return [
        # the mapping step on a survey area: 2M multibeam soundings of a
        # lawnmower track onto a 4096^2 grid at 2 m, resampled to 1 m
        _step("step_swath_2M", lines=8, pings=625, beams=400, nodes=4096, altitude=0.0),
        # a quick look at one square kilometre: the smallest scattered call
        _grid("grid_uniform_20k", "uniform", n=20000, nx=256, ny=256, dx=3.90625, radius=20.0,
              power=2.0, min_pts=3, max_pts=0),
        # one dive's swath from a deep vehicle on an odd-sized grid
        _grid("grid_swath_150k", "swath", n=150000, nx=1023, ny=769, dx=2.0, radius=6.0,
              power=3.0, min_pts=1, max_pts=16),
        # a survey with overlapping passes: far more soundings in reach of a
        # node than the cap keeps
        _grid("grid_dense_200k", "uniform", n=200000, nx=512, ny=512, dx=2.0, radius=6.0,
              power=2.0, min_pts=1, max_pts=16),
        # a cell size that is no dyadic fraction of a metre
        _grid("grid_odd_spacing", "uniform", n=120000, nx=701, ny=650, dx=3.3, radius=10.0,
              power=2.0, min_pts=2, max_pts=0),
        # nearest sounding per cell (the index grid a point editor works on)
        _nearest("nearest_500k", n=500000, nx=2048, ny=1500, dx=2.0, radius=6.0),
        # a chart's 256 uneven tiles, planned once, launched as one batch
        _batch("batch_256_tiles", tiles=256, n_lo=1000, n_hi=200000, side_hi=1024),
        # four vehicles' ping blocks into their resident grids, grids read out
        _serve("serve_4_vehicles", vehicles=4, nodes=2048, n=26000),
        # a few recorded rows filled in on board: the smallest call of all
        _resample("rows_bilinear_1e4", "bilinear", snx=100, sny=101, dnx=100, dny=100,
                  ratio_x=1.0, ratio_y=1.0, holes=0.0),
        # display zoom by a ragged factor
        _resample("zoom_bicubic_8M", "bicubic", snx=1501, sny=1300, dnx=3199, dny=2500,
                  ratio_x=0.0, ratio_y=0.0, holes=0.02),
        # a 2x chart grid by kriging with some holes in the source
        _resample("chart_kriging_16M", "kriging", snx=2048, sny=2048, dnx=4096, dny=4096,
                  ratio_x=0.0, ratio_y=0.0, holes=0.001),
        # the semivariogram a kriging range is fitted to
        _variogram("variogram_1024", nx=1024, ny=1024, dx=8.0, lags=64, holes=0.05),
    ]


def _step(name, lines, pings, beams, nodes, altitude):
    return {"name": name, "kind": "step", "lines": lines, "pings": pings, "beams": beams,
            "nodes": nodes, "altitude": altitude}


def _grid(name, pattern, n, nx, ny, dx, radius, power, min_pts, max_pts):
    return {"name": name, "kind": "grid", "pattern": pattern, "n": n, "nx": nx, "ny": ny,
            "dx": dx, "radius": radius, "power": power, "min_pts": min_pts, "max_pts": max_pts}


def _nearest(name, n, nx, ny, dx, radius):
    return {"name": name, "kind": "nearest", "n": n, "nx": nx, "ny": ny, "dx": dx,
            "radius": radius}


def _batch(name, tiles, n_lo, n_hi, side_hi):
    return {"name": name, "kind": "batch", "tiles": tiles, "n_lo": n_lo, "n_hi": n_hi,
            "side_hi": side_hi}


def _serve(name, vehicles, nodes, n):
    return {"name": name, "kind": "serve", "vehicles": vehicles, "nodes": nodes, "n": n}


def _resample(name, method, snx, sny, dnx, dny, ratio_x, ratio_y, holes):
    return {"name": name, "kind": "resample", "method": method, "snx": snx, "sny": sny,
            "dnx": dnx, "dny": dny, "ratio_x": ratio_x, "ratio_y": ratio_y, "holes": holes}


def _variogram(name, nx, ny, dx, lags, holes):
    return {"name": name, "kind": "variogram", "nx": nx, "ny": ny, "dx": dx, "lags": lags,
            "holes": holes}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: sizes spread over the logarithm of their range."""
    kind = rng.choice(["step", "grid", "grid", "grid", "nearest", "batch", "serve",
                       "resample", "resample", "variogram"])
    if kind == "step":
        # altitude 0: a surface sensor; else a deep vehicle with a narrow swath
        c = _step("", rng.randint(2, 8), _log_int(rng, 80, 600), _log_int(rng, 64, 400),
                  _log_int(rng, 300, 4000), rng.choice([0.0, 60.0, 150.0]))
    elif kind in ("grid", "nearest"):
        nx, ny = _log_int(rng, 64, 2200), _log_int(rng, 64, 2200)
        dx = rng.choice([0.5, 1.0, 2.0, 4.0, 3.90625, 3.3, 0.7])
        radius = dx * rng.choice([1.5, 2.0, 3.0, 4.0, 5.12])
        # soundings within reach of a node, on average
        reach = math.exp(rng.uniform(math.log(0.5), math.log(30.0)))
        area = (nx * dx + 2 * radius) * (ny * dx + 2 * radius)
        n = int(min(1.5e6, max(500.0, reach * area / (math.pi * radius * radius))))
        if kind == "nearest":
            c = _nearest("", n, nx, ny, dx, radius)
        else:
            cap = rng.choice([0, 0, 4, 8, 16, 16, 24])
            c = _grid("", rng.choice(["uniform", "swath"]), n, nx, ny, dx, radius,
                      rng.choice([1.0, 2.0, 2.0, 3.0, 2.5]), rng.choice([0, 1, 3]), cap)
    elif kind == "batch":
        c = _batch("", _log_int(rng, 4, 200), 1000, _log_int(rng, 5000, 200000),
                   rng.choice([128, 256, 512, 1024]))
    elif kind == "serve":
        c = _serve("", rng.randint(1, 4), _log_int(rng, 256, 2048), _log_int(rng, 2000, 50000))
    elif kind == "resample":
        method = rng.choice(["bilinear", "bicubic", "kriging"])
        snx, sny = _log_int(rng, 60, 4000), _log_int(rng, 60, 4000)
        if rng.random() < 0.3:  # rows between recorded rows
            c = _resample("", method, snx, sny + 1, snx, sny, 1.0, 1.0, rng.choice([0.0, 0.01]))
        else:
            z = rng.uniform(0.6, 2.6)
            c = _resample("", method, snx, sny, max(40, int(snx * z)), max(40, int(sny * z)),
                          0.0, 0.0, rng.choice([0.0, 0.002, 0.05]))
    else:
        c = _variogram("", _log_int(rng, 120, 1100), _log_int(rng, 120, 1100),
                       rng.choice([1.0, 4.0, 8.0]), rng.choice([16, 24, 48, 64]),
                       rng.choice([0.0, 0.05, 0.3]))
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs --

class _Sea:
    """Seeded seafloor on the GPU: 5000 m deep, six octaves of waves."""

    def __init__(self, seed):
        r = random.Random(seed * 7919 + 13)
        self.waves = []
        for o in range(6):
            k = 2.0 * math.pi / (400.0 * 2.0 ** -o * r.uniform(0.8, 1.2))
            a, t = 0.5 ** o, r.uniform(0.0, 2.0 * math.pi)
            self.waves.append((300.0 * a, k * math.cos(t), k * math.sin(t),
                               r.uniform(0.0, 2.0 * math.pi)))

    def depth(self, x, y):
        d = torch.full_like(x, 5000.0)
        for a, kx, ky, ph in self.waves:
            d += a * torch.sin(kx * x + ky * y + ph)
        return d


def _gen(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 1000003 + salt)
    return g


def _f64(*shape):
    return dict(size=shape, dtype=torch.float64, device="cuda")


def _uniform(n, w, h, margin, x0, y0, sea, g):
    x = torch.rand(generator=g, **_f64(n)) * (w + 2 * margin) - margin + x0
    y = torch.rand(generator=g, **_f64(n)) * (h + 2 * margin) - margin + y0
    return x, y, _noisy(sea, x, y, g)


def _noisy(sea, x, y, g):
    d = sea.depth(x, y)
    return -(d + torch.randn(generator=g, **_f64(x.numel())) * 0.002 * d)


def _swath(lines, pings, beams, w, h, altitude, spacing, x0, y0, sea, g):
    """Lawnmower lines along y, pings across them, beams over +-60 degrees with
    half a degree of jitter, in ping order (odd lines run back)."""
    dev = "cuda"
    xl = w / 2 + (torch.arange(lines, device=dev, dtype=torch.float64) - (lines - 1) / 2) * spacing
    py = (torch.arange(pings, device=dev, dtype=torch.float64) + 0.5) * h / pings
    py = py.expand(lines, pings).clone()
    py[1::2] = py[1::2].flip(1)
    xl = xl[:, None].expand(lines, pings)
    if altitude > 0.0:
        height = torch.full_like(py, altitude)
    else:
        height = sea.depth(xl + x0, py + y0)
    step = 120.0 / beams
    th = -60.0 + (torch.arange(beams, device=dev, dtype=torch.float64) + 0.5) * step
    th = th + torch.rand(generator=g, **_f64(lines, pings, beams)) - 0.5
    x = (xl[..., None] + height[..., None] * torch.tan(torch.deg2rad(th))).reshape(-1) + x0
    y = py[..., None].expand(lines, pings, beams).reshape(-1) + y0
    y = y.contiguous()
    return x, y, _noisy(sea, x, y, g)


def _drop_some(x, y, z, g):
    """A few soundings in a thousand are flagged invalid (NaN depth)."""
    z[torch.rand(generator=g, **_f64(z.numel())) < 0.002] = math.nan
    return x, y, z


def _soundings(c, seed):
    """Soundings and grid of a step, grid or nearest case."""
    sea, g = _Sea(seed), _gen(seed, 1)
    x0, y0 = 1000.0 * (seed % 7), -500.0 * (seed % 5)
    if c["kind"] == "step":
        w = c["nodes"] * 2.0
        spacing = 150.0 if c["altitude"] == 0.0 else w / (c["lines"] + 1)
        p = _swath(c["lines"], c["pings"], c["beams"], w, w, c["altitude"], spacing, x0, y0,
                   sea, g)
        return p, ag.make_desc(x0, y0, 2.0, 2.0, c["nodes"], c["nodes"])
    d = ag.make_desc(x0, y0, c["dx"], c["dx"], c["nx"], c["ny"])
    w, h, r = c["nx"] * c["dx"], c["ny"] * c["dx"], c["radius"]
    if c.get("pattern") == "swath":
        # as many lines as cover the width at the swath's height, pings spread
        # over the length: about n soundings in ping order
        alt = max(20.0, min(150.0, w / 4.0))
        lines = max(1, int(w / (3.0 * alt)))
        beams = 128
        pings = max(2, round(c["n"] / (lines * beams)))
        p = _swath(lines, pings, beams, w, h, alt, w / lines, x0, y0, sea, g)
    else:
        p = _uniform(c["n"], w, h, r, x0, y0, sea, g)
    return _drop_some(*p, g), d


def _idw_args(c):
    if c["kind"] == "step":
        return dict(power=2.0, radius=6.0, min_pts=1, max_pts=16)
    return dict(power=c["power"], radius=c["radius"], min_pts=c["min_pts"], max_pts=c["max_pts"])


def _tile_list(c):
    """Soundings count, side and power of each tile: the chart's layout."""
    r = random.Random(c["tiles"])
    sides = [s for s in (64, 128, 256, 512, 1024) if s <= c["side_hi"]]
    return [(_log_int(r, c["n_lo"], c["n_hi"]), r.choice(sides), float(r.randint(1, 3)))
            for _ in range(c["tiles"])]


def _tile_points(t, n, side, sea, g):
    ox, oy = (t % 16) * 4096.0, (t // 16) * 4096.0
    return _uniform(n, side * 2.0, side * 2.0, 0.0, ox, oy, sea, g), ag.make_desc(
        ox, oy, 2.0, 2.0, side, side)


def _request(c, v, seed):
    """A block of pings of vehicle v, as host arrays, and the vehicle's grid."""
    sea, g = _Sea(seed), _gen(seed, 100 + v)
    r = random.Random(seed * 17 + v)
    ext = c["nodes"] * 2.0
    x0, y0 = v * 2.0 * ext, 0.0
    beams = 400
    pings = -(-c["n"] // beams)
    alt = min(150.0, ext / 8.0)
    x, y, z = _swath(1, pings, beams, ext, 2.0 * pings, alt, 1.0, x0, y0, sea, g)
    shift = r.uniform(0.0, max(0.0, ext - 2.0 * pings))
    y += shift
    z = _noisy(sea, x, y, g)
    h = tuple(np.ascontiguousarray(a[:c["n"]].cpu().numpy()) for a in (x, y, z))
    return h, ag.make_desc(x0, y0, 2.0, 2.0, c["nodes"], c["nodes"])


def _holes(z, frac, seed):
    if frac > 0.0:
        z[torch.rand(generator=_gen(seed, 7), **_f64(*z.shape)) < frac] = math.nan
    return z


def _dem(nx, ny, dx, seed):
    """Elevations of the seafloor at the node centres, float32 [ny, nx]."""
    xs = (torch.arange(nx, device="cuda", dtype=torch.float64) + 0.5) * dx
    ys = (torch.arange(ny, device="cuda", dtype=torch.float64) + 0.5) * dx
    sea = _Sea(seed)
    z = torch.empty((ny, nx), dtype=torch.float32, device="cuda")
    for a in range(0, ny, 512):
        yy = ys[a:a + 512]
        z[a:a + 512] = -sea.depth(xs[None, :].expand(yy.numel(), nx), yy[:, None].expand(-1, nx))
    return z


def _resample_grids(c):
    """Source and destination descriptors: a ratio of 1 shifts the rows by half
    a node (infill), 0 covers the source's extent with the destination's nodes."""
    h = 4.0
    s = ag.make_desc(0.0, 0.0, h, h, c["snx"], c["sny"])
    if c["ratio_x"] == 1.0:
        d = ag.make_desc(0.0, 0.5 * h, h, h, c["dnx"], c["dny"])
    else:
        d = ag.make_desc(0.0, 0.0, h * c["snx"] / c["dnx"], h * c["sny"] / c["dny"], c["dnx"],
                         c["dny"])
    return s, d


def _out(desc, *dtypes):
    return [torch.empty((desc.ny, desc.nx), dtype=t, device="cuda") for t in dtypes]


def prepare(case, seed):
    c = case
    kind = c["kind"]
    if kind in ("step", "grid", "nearest"):
        (x, y, z), d = _soundings(c, seed)
        a = _idw_args(c) if kind != "nearest" else {"radius": c["radius"]}
        grid = ag.auv_grid_create(d)
        ws = torch.empty(ag.auv_bin_workspace_size(grid, x.numel(), a["radius"]),
                         dtype=torch.uint8, device="cuda")
        st = {"kind": kind, "grid": grid, "x": x, "y": y, "z": z, "ws": ws,
              "radius": a["radius"]}
        st["zo"], st["cnt"], st["nn"], st["nz"] = _out(d, torch.float32, torch.int32,
                                                       torch.int32, torch.float32)
        if kind != "nearest":
            st["params"] = ag.idw_params(**a)
        if kind == "step":
            st["desc"] = d
            st["up_desc"] = ag.make_desc(d.x0, d.y0, 1.0, 1.0, 2 * d.nx, 2 * d.ny)
            st["up"], = _out(st["up_desc"], torch.float32)
        return st
    if kind == "batch":
        sea, g = _Sea(seed), _gen(seed, 2)
        tiles = _tile_list(c)
        m = sum(s * s for _, s, _ in tiles)
        zo = torch.empty(m, dtype=torch.float32, device="cuda")
        nn = torch.empty(m, dtype=torch.int32, device="cuda")
        items, keep, at = [], [], 0
        for t, (n, side, p) in enumerate(tiles):
            (x, y, z), d = _tile_points(t, n, side, sea, g)
            k = side * side
            prm = ag.idw_params(power=p, radius=6.0, min_pts=1, max_pts=16)
            items.append(ag.batch_item(d, x, y, z, prm, zo[at:at + k], None, nn[at:at + k]))
            keep.append((x, y, z))
            at += k
        return {"kind": kind, "batch": ag.Batch(items), "keep": keep, "zo": zo, "nn": nn}
    if kind == "serve":
        reqs, grids = [], []
        for v in range(c["vehicles"]):
            q, d = _request(c, v, seed)
            reqs.append(q)
            grids.append(d)
        desc = ag.session_desc(grids, power=2.0, radius=6.0, min_pts=1, max_request=50000,
                               slots=8, z_ref=[-5000.0] * len(grids))
        fixed, per = ag.auv_session_budget(desc)
        arena = torch.empty(fixed + len(grids) * per, dtype=torch.uint8, device="cuda")
        return {"kind": kind, "session": ag.Session(desc, arena), "requests": reqs}
    if kind == "resample":
        s, d = _resample_grids(c)
        dst, = _out(d, torch.float32)
        return {"kind": kind, "method": c["method"], "s": s, "d": d, "dst": dst,
                "src": _holes(_dem(s.nx, s.ny, s.dx, seed), c["holes"], seed),
                "range": 3.0 * s.dx}
    if kind == "variogram":
        z = _holes(_dem(c["nx"], c["ny"], c["dx"], seed), c["holes"], seed)
        return {"kind": kind, "src": z, "lags": c["lags"],
                "desc": ag.make_desc(0.0, 0.0, c["dx"], c["dx"], c["nx"], c["ny"])}
    raise ValueError(kind)


# --------------------------------------------------------------------- run --

def run(state):
    s = state
    kind = s["kind"]
    if kind in ("step", "grid", "nearest"):
        bins = ag.auv_bin_points(s["grid"], s["x"], s["y"], s["z"], s["radius"], ws=s["ws"])
        if kind == "nearest":
            ag.auv_interp_nearest(s["grid"], bins, s["radius"], s["nn"], s["nz"])
            return {"nn_idx": s["nn"], "nn_z": s["nz"]}
        if kind == "step":
            ag.auv_interp_idw(s["grid"], bins, s["params"], s["zo"], None, s["nn"], s["nz"])
            ag.auv_resample_bilinear(s["zo"], s["desc"], s["up"], s["up_desc"])
            return {"z": s["zo"], "nn_idx": s["nn"], "nn_z": s["nz"], "up": s["up"]}
        ag.auv_interp_idw(s["grid"], bins, s["params"], s["zo"], s["cnt"], s["nn"], s["nz"])
        return {"z": s["zo"], "cnt": s["cnt"], "nn_idx": s["nn"], "nn_z": s["nz"]}
    if kind == "batch":
        s["batch"].launch()
        return {"z": s["zo"], "nn_idx": s["nn"]}
    if kind == "serve":
        ses = s["session"]
        for v, (x, y, z) in enumerate(s["requests"]):
            ses.submit(v, x, y, z)
        ses.drain()
        return {"grids": [ses.read_grid(v) for v in range(len(s["requests"]))]}
    if kind == "resample":
        if s["method"] == "bilinear":
            ag.auv_resample_bilinear(s["src"], s["s"], s["dst"], s["d"])
        elif s["method"] == "bicubic":
            ag.auv_resample_bicubic(s["src"], s["s"], s["dst"], s["d"])
        else:
            ag.auv_resample_kriging(s["src"], s["s"], s["dst"], s["d"], s["range"])
        return {"dst": s["dst"]}
    gx, gy, px, py = ag.auv_variogram(s["src"], s["desc"], s["lags"])
    return {"gamma_x": gx, "gamma_y": gy, "pairs_x": px, "pairs_y": py}


# -------------------------------------------------------------------- work --

def work(case):
    """Inputs read once, outputs written once; operations of the selected
    (node, sounding) pairs, about ten each, or of the stencil."""
    c = case
    kind = c["kind"]

    def scattered(n, nx, ny, dx, radius, cap, out_bytes):
        m = nx * ny
        reach = n * math.pi * radius * radius / ((nx * dx + 2 * radius) * (ny * dx + 2 * radius))
        pairs = m * (min(reach, cap) if cap else reach)
        return {"bytes": 24.0 * n + out_bytes * m, "flops": 10.0 * pairs}

    if kind == "step":
        n, m = c["lines"] * c["pings"] * c["beams"], c["nodes"]
        w = scattered(n, m, m, 2.0, 6.0, 16, 12)
        return {"bytes": w["bytes"] + 4.0 * m * m * 5, "flops": w["flops"] + 36.0 * m * m}
    if kind == "grid":
        return scattered(c["n"], c["nx"], c["ny"], c["dx"], c["radius"], c["max_pts"], 16)
    if kind == "nearest":
        return scattered(c["n"], c["nx"], c["ny"], c["dx"], c["radius"], 1, 8)
    if kind == "batch":
        ws = [scattered(n, s, s, 2.0, 6.0, 16, 8) for n, s, _ in _tile_list(c)]
        return {k: sum(w[k] for w in ws) for k in ("bytes", "flops")}
    if kind == "serve":
        m = c["nodes"] ** 2
        # the request in, the touched nodes' sums updated, the grid read out
        # (five sums in, depth and count out)
        touched = min(m, c["n"] / 400.0 * 300.0 / 2.0)
        return {"bytes": c["vehicles"] * (24.0 * c["n"] + 40.0 * touched + 28.0 * m),
                "flops": c["vehicles"] * 280.0 * c["n"]}
    if kind == "resample":
        per = {"bilinear": 9.0, "bicubic": 50.0, "kriging": 130.0}[c["method"]]
        d = c["dnx"] * c["dny"]
        return {"bytes": 4.0 * (c["snx"] * c["sny"] + d), "flops": per * d}
    m = c["nx"] * c["ny"]
    return {"bytes": 4.0 * m + 32.0 * c["lags"], "flops": 2.0 * 4.0 * c["lags"] * m}


# ------------------------------------------------------------------- exact --

def _node_lattice(n, d):
    return torch.round((torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) * d
                       * _LATTICE).to(torch.int64)


def _exact_idw(x, y, z, d, radius, power=2.0, min_pts=1, max_pts=0, nearest_only=False):
    """IDW and nearest depth in 64 bits: every (sounding, node) pair within the
    radius, ranked by (squared lattice distance, index) where a cap cuts."""
    R = round(radius * _LATTICE)
    Xn, Yn = _node_lattice(d.nx, d.dx), _node_lattice(d.ny, d.dy)
    keep = torch.isfinite(x) & torch.isfinite(y) & torch.isfinite(z)
    orig = torch.nonzero(keep).reshape(-1)
    x, y, z = x[orig] - d.x0, y[orig] - d.y0, z[orig]
    wx, wy = int(2 * radius / d.dx) + 3, int(2 * radius / d.dy) + 3
    nodes, dist, who, wts = [], [], [], []
    step = max(1, 30_000_000 // (wx * wy))
    for a in range(0, x.numel(), step):
        xs, ys = x[a:a + step], y[a:a + step]
        X = torch.round(xs * _LATTICE).to(torch.int64)
        Y = torch.round(ys * _LATTICE).to(torch.int64)
        jb = torch.floor((xs - radius) / d.dx - 0.5).to(torch.int64)
        ja = torch.floor((ys - radius) / d.dy - 0.5).to(torch.int64)
        cb = jb[:, None] + torch.arange(wx, device="cuda")
        ca = ja[:, None] + torch.arange(wy, device="cuda")
        inb, ina = (cb >= 0) & (cb < d.nx), (ca >= 0) & (ca < d.ny)
        cb, ca = cb.clamp(0, d.nx - 1), ca.clamp(0, d.ny - 1)
        D = ((X[:, None] - Xn[cb]) ** 2)[:, None, :] + ((Y[:, None] - Yn[ca]) ** 2)[:, :, None]
        i, r, q = torch.nonzero((D <= R * R) & inb[:, None, :] & ina[:, :, None], as_tuple=True)
        b, e = cb[i, q], ca[i, r]
        nodes.append((e * d.nx + b).to(torch.int32))
        dist.append(D[i, r, q])
        who.append((i + a).to(torch.int32))
        fx, fy = xs[i] - (b + 0.5) * d.dx, ys[i] - (e + 0.5) * d.dy
        wts.append(fx * fx + fy * fy)
        del D, i, r, q, b, e, fx, fy
    m = d.nx * d.ny
    if not nodes:
        nodes, dist, who, wts = ([torch.zeros(0, dtype=t, device="cuda")] for t in (
            torch.int32, torch.int64, torch.int32, torch.float64))
    node, D, i, f2 = (torch.cat(v) for v in (nodes, dist, who, wts))
    del nodes, dist, who, wts
    # by node, then (distance, index): the pairs come by ascending index
    o = torch.sort(D, stable=True).indices
    o = o[torch.sort(node[o], stable=True).indices]
    node, D, i, f2 = node[o].long(), D[o], i[o].long(), f2[o]
    cnt = torch.bincount(node, minlength=m)
    start = torch.cumsum(cnt, 0) - cnt
    nz = torch.full((m,), math.nan, dtype=torch.float64, device="cuda")
    some = cnt > 0
    nz[some] = z[i[start[some]]]
    if nearest_only:
        return None, nz.reshape(d.ny, d.nx)
    if max_pts:
        rank = torch.arange(node.numel(), device="cuda") - start[node]
        sel = rank < max_pts
        node, D, i, f2 = node[sel], D[sel], i[sel], f2[sel]
        cnt = cnt.clamp(max=max_pts)
    hit = D == 0
    hits = torch.bincount(node[hit], minlength=m)
    wt = torch.where(hits[node] > 0, hit.double(), f2.clamp(min=1e-300) ** (-0.5 * power))
    ref = nz[node]
    num = torch.zeros(m, dtype=torch.float64, device="cuda").index_add_(0, node, wt * (z[i] - ref))
    den = torch.zeros(m, dtype=torch.float64, device="cuda").index_add_(0, node, wt)
    v = nz + num / den
    v[(hits == 0) & ((cnt == 0) | (cnt < min_pts))] = math.nan
    return v.reshape(d.ny, d.nx), nz.reshape(d.ny, d.nx)


def _axis(d0, dd, n, s0, ds, ns):
    u = (d0 + (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) * dd - s0) / ds - 0.5
    u = u.clamp(0.0, float(ns - 1))
    i0 = torch.floor(u)
    return u, i0.long(), (i0.long() + 1).clamp(max=ns - 1), u - i0


def _exact_bilinear(src, s, d):
    _, i0, i1, t = _axis(d.x0, d.dx, d.nx, s.x0, s.dx, s.nx)
    _, j0, j1, u = _axis(d.y0, d.dy, d.ny, s.y0, s.dy, s.ny)
    out = torch.empty((d.ny, d.nx), dtype=torch.float64, device="cuda")
    for a in range(0, d.ny, 512):
        p, q = src[j0[a:a + 512]].double(), src[j1[a:a + 512]].double()
        top = p[:, i0] + t * (p[:, i1] - p[:, i0])
        bot = q[:, i0] + t * (q[:, i1] - q[:, i0])
        out[a:a + 512] = top + u[a:a + 512, None] * (bot - top)
    return out


def _cubic(p, t):
    a, b, c, e = p
    return 0.5 * (2 * b + t * (c - a + t * (2 * a - 5 * b + 4 * c - e
                                            + t * (3 * (b - c) + e - a))))


def _exact_bicubic(src, s, d):
    _, i0, _, t = _axis(d.x0, d.dx, d.nx, s.x0, s.dx, s.nx)
    _, j0, _, u = _axis(d.y0, d.dy, d.ny, s.y0, s.dy, s.ny)
    out = _exact_bilinear(src, s, d)
    for a in range(0, d.ny, 256):
        rows = []
        for k in range(-1, 3):
            r = src[(j0[a:a + 256] + k).clamp(0, s.ny - 1)].double()
            rows.append(_cubic([r[:, (i0 + q).clamp(0, s.nx - 1)] for q in range(-1, 3)], t))
        v = _cubic(rows, u[a:a + 256, None])
        out[a:a + 256] = torch.where(torch.isfinite(v), v, out[a:a + 256])
    return out


def _exact_kriging(src, s, d, rng):
    out = _exact_bilinear(src, s, d)
    if s.nx < 5 or s.ny < 5:
        return out
    q = torch.arange(25, device="cuda")
    qx, qy = (q % 5).double() * s.dx, (q // 5).double() * s.dy
    K = torch.ones((26, 26), dtype=torch.float64, device="cuda")
    K[25, 25] = 0.0
    K[:25, :25] = -torch.expm1(-torch.hypot(qx[:, None] - qx, qy[:, None] - qy) / rng)
    inv = torch.linalg.inv(K.cpu()).cuda()
    ux, _, _, _ = _axis(d.x0, d.dx, d.nx, s.x0, s.dx, s.nx)
    uy, _, _, _ = _axis(d.y0, d.dy, d.ny, s.y0, s.dy, s.ny)
    bx = (torch.floor(ux + 0.5).long() - 2).clamp(0, s.nx - 5)
    by = (torch.floor(uy + 0.5).long() - 2).clamp(0, s.ny - 5)
    ex = (ux - bx)[None, :] * s.dx
    for a in range(0, d.ny, 128):
        rows = by[a:a + 128]
        ey = (uy[a:a + 128] - rows)[:, None] * s.dy
        zc = src[rows + 2].double()[:, bx + 2]
        g = torch.stack([-torch.expm1(-torch.hypot(ex - qx[k], ey - qy[k]) / rng)
                         for k in range(25)] + [torch.ones_like(zc)])
        lam = torch.tensordot(inv, g, dims=([1], [0]))
        v = zc.clone()
        for k in range(25):
            v += lam[k] * (src[rows + k // 5].double()[:, bx + k % 5] - zc)
        out[a:a + 128] = torch.where(torch.isfinite(v), v, out[a:a + 128])
    return out


def _exact_variogram(z, lags):
    z = z.double()
    ok = torch.isfinite(z)
    gam, num = ([], []), ([], [])
    for axis in (1, 0):
        for k in range(1, lags + 1):
            n = max(0, z.shape[axis] - k)
            a, b = z.narrow(axis, 0, n), z.narrow(axis, z.shape[axis] - n, n)
            both = ok.narrow(axis, 0, n) & ok.narrow(axis, z.shape[axis] - n, n)
            e = torch.where(both, a - b, torch.zeros_like(a))
            c = int(both.sum())
            gam[1 - axis].append(float((e * e).sum()) / (2 * c) if c else math.nan)
            num[1 - axis].append(c)
    return {"gamma_x": np.array(gam[0]), "gamma_y": np.array(gam[1]),
            "pairs_x": np.array(num[0], dtype=np.int64),
            "pairs_y": np.array(num[1], dtype=np.int64)}


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind in ("step", "grid"):
        (x, y, z), d = _soundings(c, seed)
        v, nz = _exact_idw(x, y, z, d, **_idw_args(c))
        if kind == "grid":
            return {"z": v, "cnt": None, "nn_idx": None, "nn_z": nz}
        up = ag.make_desc(d.x0, d.y0, 1.0, 1.0, 2 * d.nx, 2 * d.ny)
        return {"z": v, "nn_idx": None, "nn_z": nz, "up": _exact_bilinear(v, d, up)}
    if kind == "nearest":
        (x, y, z), d = _soundings(c, seed)
        return {"nn_idx": None,
                "nn_z": _exact_idw(x, y, z, d, c["radius"], nearest_only=True)[1]}
    if kind == "batch":
        sea, g = _Sea(seed), _gen(seed, 2)
        out = []
        for t, (n, side, p) in enumerate(_tile_list(c)):
            (x, y, z), d = _tile_points(t, n, side, sea, g)
            out.append(_exact_idw(x, y, z, d, 6.0, p, 1, 16)[0].reshape(-1))
        return {"z": torch.cat(out), "nn_idx": None}
    if kind == "serve":
        out = []
        for v in range(c["vehicles"]):
            q, d = _request(c, v, seed)
            z, _ = _exact_idw(*(torch.from_numpy(a).cuda() for a in q), d, 6.0)
            out.append((z, None))
        return {"grids": out}
    if kind == "resample":
        s, d = _resample_grids(c)
        src = _holes(_dem(s.nx, s.ny, s.dx, seed), c["holes"], seed)
        if c["method"] == "bilinear":
            return {"dst": _exact_bilinear(src, s, d)}
        if c["method"] == "bicubic":
            return {"dst": _exact_bicubic(src, s, d)}
        return {"dst": _exact_kriging(src, s, d, 3.0 * s.dx)}
    z = _holes(_dem(c["nx"], c["ny"], c["dx"], seed), c["holes"], seed)
    return _exact_variogram(z, c["lags"])
