"""The work a user of this library has it do, as measurable cases.

Each case is one call (or one short sequence of calls) through the public entry
points of paper_2601_20758_amd on synthetic clustered clouds: a node grid
evaluated over a region of a resident cloud, a cloud opened and shown, the
adaptive estimator, a batch and a served second of requests, and the
consumers of a grid. Clouds hold 20% uniform background and 80% in 2,000
Gaussian clumps of power-law mass, like the clouds the tests and the benchmark
use, drawn on the GPU from the seed; regions smaller than the cloud sit around
one of its ten most massive clumps, where users zoom in.
"""
import math

import numpy as np
import torch

import paper_2601_20758_amd as sfk

H0 = 0.01            # bandwidth as a fraction of a region's side (zooms, batches, traces)
N_CLUMPS = 2000
DRAW_CHUNK = 1 << 25
EXACT_PAIRS = 6e9    # (particle, node offset) tests an exact grid may take


class Region:
    """One region-of-interest request, with the fields the binding reads."""

    def __init__(self, lo, hi, res, kernel, bw, h, norm="paper", set="cloud"):
        self.lo, self.hi, self.res = tuple(lo), tuple(hi), tuple(int(r) for r in res)
        self.kernel, self.bw, self.h, self.norm, self.set, self.tag = kernel, bw, tuple(h), norm, set, 0

    @property
    def n_nodes(self):
        return self.res[0] * self.res[1] * self.res[2]


# ---------------------------------------------------------------- the cases

def _case(name, kind, points, side=1.0, res=(64, 64, 64), kernel="epanechnikov", bw="roi_scaled",
          h=H0, norm="paper", set="cloud", knn=0, count=1):
    c = {"kind": kind, "points": points, "side": side, "rx": res[0], "ry": res[1], "rz": res[2],
         "kernel": kernel, "bw": bw, "h": h, "norm": norm, "set": set, "knn": knn, "count": count}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a preview grid of a small cloud, where launches and latency are all
        _case("preview_20k", "grid", 20_000, res=(32, 32, 32), bw="fixed", h=0.02),
        # the estimator on a cloud of the size published studies use, at their 64^3 grid:
        # the recomputation behind one step of an interactive session
        _case("adaptive_442k", "grid", 442_000, side=0.5, res=(64, 64, 64), bw="mbe", set="in_roi"),
        # the same estimator at a fine grid inside a dense clump of a large cloud
        _case("adaptive_100m", "grid", 100_000_000, side=0.05, res=(128, 128, 128), bw="mbe", set="in_roi"),
        # the per-point analysis step: neighbour bandwidths of a whole cloud and its Gaussian field
        _case("point_step_10m", "open", 10_000_000, res=(128, 128, 128), kernel="gauss_trunc3",
              bw="per_point", knn=32),
        # a resident cloud whose bandwidths are known, on a ragged grid
        _case("point_grid_1m", "grid", 1_000_003, side=0.8, res=(101, 87, 93), bw="per_point", norm="count"),
        # opening a cloud: the index is built and the first overview grid drawn
        _case("open_10m", "open", 10_000_019, res=(64, 64, 64)),
        # a uniform truncated Gaussian with one length per axis, ragged grid
        _case("gauss_10m", "grid", 10_000_000, res=(96, 80, 112), kernel="gauss_trunc3", bw="fixed",
              h=0.004, norm="count"),
        # the finest overview of a large cloud, and the same grid deep inside a clump
        _case("overview_100m", "grid", 100_000_000, res=(256, 256, 256)),
        _case("zoom_100m", "grid", 100_000_000, side=1.0 / 64, res=(256, 256, 256)),
        # many uneven regions at once (sides and grids spread over their ranges)
        _case("batch_100m", "batch", 100_000_000, count=256),
        # one second of requests of 8 viewers at 90 Hz, all waiting, on a billion points
        _case("serve_1b", "serve", 1_000_000_000, count=720),
        # what follows a grid: density at every particle, the points above a threshold, the surface
        _case("consume_10m", "consume", 10_000_000, res=(128, 128, 128)),
    ]


def _log(rng, a, b):
    return math.exp(rng.uniform(math.log(a), math.log(b)))


def draw(rng):
    kind = rng.choice(["grid", "grid", "grid", "grid", "point", "point", "mbe", "mbe", "open", "open",
                       "batch", "consume", "serve"])
    norm = rng.choice(["paper", "count"])
    r = _log(rng, 16, 256)
    res = tuple(max(2, int(r * rng.uniform(0.7, 1.0))) for _ in range(3))
    if kind == "grid":
        points = int(_log(rng, 2e4, 1e8))
        kernel = rng.choice(["epanechnikov", "epanechnikov", "gauss_trunc3"])
        side = rng.choice([1.0, _log(rng, 1e-3, 1.0)])
        h = min(_log(rng, 0.004, 0.03), 3.4 / max(res)) / (3.0 if kernel == "gauss_trunc3" else 1.0)
        return _case("", "grid", points, side, res, kernel, "roi_scaled", h, norm,
                     rng.choice(["cloud", "cloud", "cloud", "in_roi"]) if points < 2e7 else "cloud")
    if kind == "point":
        points = int(_log(rng, 2e4, 1e7))
        res = tuple(min(v, 140) for v in res)
        knn = rng.choice([0, 8, 16, 24, 32])
        return _case("", "open" if knn else "grid", points, 1.0 if knn else _log(rng, 0.3, 1.0), res,
                     rng.choice(["epanechnikov", "gauss_trunc3"]), "per_point", 0.0, norm, "cloud", knn)
    if kind == "mbe":
        res = tuple(min(v, 140) for v in res)
        return _case("", "grid", int(_log(rng, 7e4, 1e8)), _log(rng, 0.02, 0.3), res, bw="mbe",
                     norm=norm, set="in_roi")
    if kind == "open":
        res = tuple(min(v, 128) for v in res)
        return _case("", "open", int(_log(rng, 2e4, 5e7)), 1.0, res, norm=norm)
    if kind == "batch":
        return _case("", "batch", int(_log(rng, 1e6, 1e8)), count=int(_log(rng, 8, 256)), norm=norm)
    if kind == "consume":
        return _case("", "consume", int(_log(rng, 1e5, 2e7)), _log(rng, 0.1, 1.0), res, norm=norm)
    return _case("", "serve", int(_log(rng, 1e7, 3e8)), count=int(_log(rng, 60, 720)))


# ------------------------------------------------------------------- inputs

_context = None


def _ctx():
    """The program's one context."""
    global _context
    if _context is None:
        _context = sfk.Context(0)
    return _context


def _cloud(n, seed):
    """((n, 3) float32 points on the GPU, centres of the ten most massive clumps)."""
    g = np.random.default_rng(seed)
    u = g.random(N_CLUMPS)
    mass = (1.0 + u * (1e3 ** -0.8 - 1.0)) ** (-1.0 / 0.8)
    centre = g.uniform(0.05, 0.95, (N_CLUMPS, 3))
    width = (0.02 * (mass / 1e3) ** (1 / 3))[:, None] * np.concatenate(
        [np.ones((N_CLUMPS, 1)), g.uniform(0.3, 1.0, (N_CLUMPS, 2))], axis=1)
    turn = np.linalg.qr(g.standard_normal((N_CLUMPS, 3, 3)))[0]
    n_back = n // 5
    count = g.multinomial(n - n_back, mass / mass.sum())
    dev = torch.device("cuda")
    tg = torch.Generator(device=dev)
    tg.manual_seed(int(seed))
    out = torch.empty((n, 3), dtype=torch.float32, device=dev)
    for a in range(0, n_back, DRAW_CHUNK):
        b = min(n_back, a + DRAW_CHUNK)
        out[a:b] = torch.rand((b - a, 3), generator=tg, device=dev)
    c_d = torch.as_tensor(centre, dtype=torch.float32, device=dev)
    axes = torch.as_tensor(turn * width[:, None, :], dtype=torch.float32, device=dev)
    ends = torch.as_tensor(np.cumsum(count), device=dev)
    for a in range(0, n - n_back, DRAW_CHUNK):
        b = min(n - n_back, a + DRAW_CHUNK)
        ids = torch.searchsorted(ends, torch.arange(a, b, device=dev), right=True)
        z = torch.randn((b - a, 3), generator=tg, device=dev)
        p = c_d[ids]
        ax = axes[ids]
        for k in range(3):
            p += ax[:, :, k] * z[:, k:k + 1]
        out[n_back + a:n_back + b] = p - torch.floor(p)  # the box is periodic
        del ids, z, p, ax
    return out, centre[np.argsort(-mass)[:10]]


def _box(centre, side):
    if side >= 1.0:
        return (0.0, 0.0, 0.0), (1.0, 1.0, 1.0)
    c = np.clip(centre, side / 2, 1 - side / 2)
    return tuple(float(v) for v in c - side / 2), tuple(float(v) for v in c + side / 2)


def _regions(case, seed, tops):
    g = np.random.default_rng([seed, 1])
    shape = np.random.default_rng(case["count"])  # sides and grids are the case's, places the seed's
    if case["kind"] == "batch":
        # sides and grids as the benchmark's batch: anywhere in the cloud
        out = []
        for _ in range(case["count"]):
            s = math.exp(shape.uniform(math.log(1e-3), 0.0))
            r = int(shape.integers(16, 129))
            lo, hi = _box(g.uniform(s / 2, 1 - s / 2, 3), s)
            out.append(Region(lo, hi, (r, r, r), "epanechnikov", "roi_scaled", (H0,) * 3, case["norm"]))
        return out
    if case["kind"] == "serve":
        # eight viewers, each panning from its last centre
        centre = g.uniform(0, 1, (8, 3))
        out = []
        for i in range(case["count"]):
            s = math.exp(shape.uniform(math.log(1e-4), 0.0))
            v = i % 8
            centre[v] = np.clip(centre[v] + g.normal(0, 0.25 * s, 3), s / 2, 1 - s / 2)
            r = int(shape.choice((32, 48, 64, 96, 128)))
            lo, hi = _box(centre[v], s)
            out.append(Region(lo, hi, (r, r, r), "epanechnikov", "roi_scaled", (H0,) * 3))
        return out
    lo, hi = _box(tops[int(g.integers(0, len(tops)))], case["side"])
    h = (case["h"],) * 3
    if case["bw"] == "fixed":  # one length per axis
        h = (case["h"], case["h"] * 1.25, case["h"] * 0.8)
    return [Region(lo, hi, (case["rx"], case["ry"], case["rz"]), case["kernel"], case["bw"], h,
                   case["norm"], case["set"])]


def _lengths(pts, seed):
    """Per-point bandwidths of a cloud whose owner knows them: a few mean spacings, uneven."""
    tg = torch.Generator(device=pts.device)
    tg.manual_seed(int(seed) + 7)
    u = torch.rand(pts.shape[0], generator=tg, device=pts.device)
    return (0.6 + 1.2 * u) * (2.0 / pts.shape[0] ** (1 / 3))


def _counts(pts, r):
    """The grid in hand where a grid is consumed: points per node, smoothed over 3^3 nodes."""
    m = torch.zeros(r.n_nodes, dtype=torch.int64, device=pts.device)
    for a in range(0, pts.shape[0], DRAW_CHUNK):
        p = pts[a:a + DRAW_CHUNK]
        p = p[_inside(p, r)]
        i = [torch.round((p[:, k].double() - r.lo[k]) * (r.res[k] - 1) / (r.hi[k] - r.lo[k])).long()
             for k in range(3)]
        m += torch.bincount(i[0] + r.res[0] * (i[1] + r.res[1] * i[2]), minlength=r.n_nodes)
    g = m.double().view(1, 1, r.res[2], r.res[1], r.res[0])
    g = torch.nn.functional.avg_pool3d(g, 3, stride=1, padding=1)
    return g.float().view(-1)


def prepare(case, seed):
    ctx = _ctx()
    pts, tops = _cloud(case["points"], seed)
    rois = _regions(case, seed, tops)
    st = {"case": case, "ctx": ctx, "rois": rois}
    sizes = [r.n_nodes for r in rois]
    st["out"] = torch.zeros(sum(sizes), device="cuda")
    st["outs"] = list(torch.split(st["out"], sizes))
    if case["kind"] == "open":
        st["pts"] = pts
        return st
    if case["kind"] == "consume":
        st["pts"] = pts
        st["out"] = _counts(pts, rois[0])
        st["iso"] = float(st["out"].mean()) * 2.0
        # what the program keeps of a selection and a surface, at their largest
        st["selected"] = torch.zeros(case["points"], dtype=torch.int64, device="cuda")
        st["surface"] = torch.zeros((2 * rois[0].n_nodes, 3, 3), device="cuda")
        return st
    per_point = case["bw"] == "per_point"
    st["tree"] = ctx.build_tree(pts, h=_lengths(pts, seed) if per_point else None)
    return st


def run(st):
    ctx, case, rois = st["ctx"], st["case"], st["rois"]
    kind = case["kind"]
    if kind == "open":
        tree = ctx.build_tree(st["pts"], knn_k=case["knn"])
        out = ctx.eval_roi(tree, rois[0], out=st["out"])
        tree.close()
        return out
    if kind == "batch":
        ctx.wait(ctx.submit(st["tree"], rois, st["outs"]))
        return st["out"]
    if kind == "serve":
        ctx.serve(st["tree"], [0.0] * len(rois), rois, st["outs"], mode=0, n_slots=4, max_batch=64)
        return st["out"]
    if kind == "consume":
        r, grid, iso = rois[0], st["out"], st["iso"]
        density = ctx.sample_density(r, grid, st["pts"])
        sel = ctx.select_points(r, grid, iso, st["pts"])
        st["selected"][:sel.numel()].copy_(sel)
        tri = ctx.iso_surface(r, grid, iso)
        st["surface"][:tri.shape[0]].copy_(tri)
        return {"density": density, "selected": st["selected"], "surface": st["surface"]}
    return ctx.eval_roi(st["tree"], rois[0], out=st["out"])


# --------------------------------------------------------------------- work

def _share(case, side):
    """About the part of a cloud in a region of this side around a massive clump."""
    return 1.0 if side >= 1.0 else min(1.0, side ** 3 + 0.02 * min(1.0, side / 0.08) ** 3)


def work(case):
    """Bytes: the particles the regions reach (12 B each) and the grids written (4 B a
    node). Operations: per particle and node inside its support 9 (Epanechnikov) or 14
    (truncated Gaussian); per particle 8 for each of its k neighbours found."""
    n, kind = case["points"], case["kind"]
    ops = 14.0 if case["kernel"] == "gauss_trunc3" else 9.0
    m = case["rx"] * case["ry"] * case["rz"]
    if kind in ("batch", "serve"):
        lo, hi, nodes = (1e-3, 1.0, 72.0 ** 3 * 1.5) if kind == "batch" else (1e-4, 1.0, 5.5e5)
        share = 1.0 / (3.0 * math.log(hi / lo))  # mean of side^3, sides log-uniform
        sup = 4.19 * (H0 * 80) ** 3
        return {"bytes": case["count"] * (12.0 * n * share + 4.0 * nodes),
                "flops": ops * case["count"] * n * share * sup}
    if kind == "consume":
        return {"bytes": 2 * 12.0 * n + 4.0 * n + 8.0 * n * 0.5 + 8.0 * m, "flops": 48.0 * n + 8.0 * m}
    n_in = n * _share(case, case["side"])
    reach = 3.0 if case["kernel"] == "gauss_trunc3" else 1.0
    rel = case["h"] if case["bw"] == "roi_scaled" else case["h"] / case["side"]
    if case["bw"] == "per_point":
        rel = 1.5 * (32.0 / 200.0 / n) ** (1 / 3) / case["side"]
    if case["bw"] == "mbe":
        rel = 2.0 / max(case["rx"], 2)
    sup = 4.19 * (reach * rel) ** 3 * m
    return {"bytes": 12.0 * (n if kind == "open" else n_in) + 4.0 * m,
            "flops": ops * n_in * sup + 8.0 * n * case["knn"]}


# ------------------------------------------------------- the results in 64 bits

def _ck(kernel):
    if kernel == "epanechnikov":
        return 15.0 / (8.0 * math.pi)
    p = math.erf(3.0 / math.sqrt(2.0)) - math.sqrt(2.0 / math.pi) * 3.0 * math.exp(-4.5)
    return 1.0 / ((2.0 * math.pi) ** 1.5 * p)


def _field(pts, ih, w, r, kernel):
    """sum_j w_j K(u_j) at every node of r, in 64 bits; ih (3,) or (n, 3), w a number or (n,).
    None where it would take too long."""
    reach = 3.0 if kernel == "gauss_trunc3" else 1.0
    dev = pts.device
    lo = torch.tensor(r.lo, dtype=torch.float64, device=dev)
    hi = torch.tensor(r.hi, dtype=torch.float64, device=dev)
    res = torch.tensor(r.res, device=dev)
    s = (hi - lo) / (res - 1)
    grid = torch.zeros(r.n_nodes, dtype=torch.float64, device=dev)
    parts, cost = [], 0.0
    for a in range(0, pts.shape[0], 1 << 24):
        p = pts[a:a + (1 << 24)].double()
        i = ih if ih.dim() == 1 else ih[a:a + (1 << 24)]
        half = reach / i.double() / s + 1e-6
        f = (p - lo) / s
        first = torch.clamp(torch.ceil(f - half), min=0)
        last = torch.minimum(torch.floor(f + half), (res - 1).double())
        keep = (first <= last).all(1).nonzero().squeeze(1) + a
        if keep.numel():
            wide = (last - first).amax(1)[keep - a].int() + 1
            parts.append((keep, wide))
            cost += float((wide.double() ** 3).sum())
        if cost > EXACT_PAIRS:
            return None
    if not parts:
        return grid
    keep, wide = (torch.cat(v) for v in zip(*parts))
    wide, order = torch.sort(wide)
    keep = keep[order]
    a = 0
    while a < keep.numel():
        b = min(keep.numel(), a + (1 << 21))
        span = int(wide[b - 1])
        ids = keep[a:b]
        p = pts[ids].double()
        i = (ih if ih.dim() == 1 else ih[ids]).double()
        ww = w if not torch.is_tensor(w) else w[ids]
        half = reach / i / s + 1e-6
        first = torch.clamp(torch.ceil((p - lo) / s - half), min=0).long()
        sq, at, ok = [], [], []
        for d in range(span):
            n = first + d
            x = lo + (n.double() * (hi - lo)) / (res - 1)
            u = (x - p) * i
            sq.append(u * u)
            at.append(n)
            ok.append(n < res)
        for dx in range(span):
            for dy in range(span):
                sxy = sq[dx][:, 0] + sq[dy][:, 1]
                oxy = ok[dx][:, 0] & ok[dy][:, 1]
                for dz in range(span):
                    u2 = sxy + sq[dz][:, 2]
                    m = oxy & ok[dz][:, 2] & (u2 < reach * reach)
                    v = torch.exp(-0.5 * u2) if reach > 1.0 else 1.0 - u2
                    v = torch.where(m, v * ww, torch.zeros_like(v))
                    idx = at[dx][:, 0] + r.res[0] * (at[dy][:, 1] + r.res[1] * at[dz][:, 2])
                    grid.index_add_(0, torch.where(m, idx, torch.zeros_like(idx)), v)
        a = b
    return grid


def _neighbour_h2(pts, k):
    """Squared distance to the k-th nearest other point (float32 operations, as defined)."""
    n = pts.shape[0]
    out = torch.empty(n, dtype=torch.float32, device=pts.device)
    step = max(1, (1 << 27) // n)
    for a in range(0, n, step):
        q = pts[a:a + step]
        d = [q[:, None, j] - pts[None, :, j] for j in range(3)]
        d2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]
        i = torch.arange(q.shape[0], device=pts.device)
        d2[i, a + i] = math.inf
        out[a:a + step] = torch.topk(d2, k, dim=1, largest=False).values[:, k - 1]
    return out


def _trilinear(grid, r, pts):
    """The 64-bit trilinear value of a node grid at points of its closed box."""
    c, t = [], []
    for k in range(3):
        f = (pts[:, k].double() - r.lo[k]) * (r.res[k] - 1) / (r.hi[k] - r.lo[k])
        i = torch.clamp(torch.floor(f).long(), 0, r.res[k] - 2)
        c.append(i)
        t.append(torch.clamp(f - i, 0.0, 1.0))
    v = torch.zeros(pts.shape[0], dtype=torch.float64, device=pts.device)
    for b in range(8):
        d = (b & 1, (b >> 1) & 1, b >> 2)
        wt = torch.ones_like(v)
        for k in range(3):
            wt = wt * (t[k] if d[k] else 1.0 - t[k])
        v += wt * grid[(c[0] + d[0]) + r.res[0] * ((c[1] + d[1]) + r.res[1] * (c[2] + d[2]))].double()
    return v


def _inside(pts, r):
    p = pts.double()
    return ((p >= torch.tensor(r.lo, dtype=torch.float64, device=pts.device)) &
            (p <= torch.tensor(r.hi, dtype=torch.float64, device=pts.device))).all(1)


def _adaptive(pts, r):
    """The modified Breiman estimator of the particles in the region's box."""
    b = pts[_inside(pts, r)]
    n = b.shape[0]
    if n < 2:
        return None
    s = [(r.hi[k] - r.lo[k]) / (r.res[k] - 1) for k in range(3)]
    ell = []
    for k in range(3):
        x = torch.sort(b[:, k].double()).values

        def at(q):
            pos = (n - 1) * q
            i = min(int(pos), n - 2)
            return float(x[i]) + (pos - i) * (float(x[i + 1]) - float(x[i]))

        v = 2.0 * (at(0.8) - at(0.2)) / math.log(n)
        ell.append(np.float32(v if v > 0.0 else 5.0 * s[k]))
    scale = _ck("epanechnikov") * (1.0 if r.norm == "count" else 1.0 / n)
    ih = torch.tensor([1.0 / float(v) for v in ell], dtype=torch.float32, device=pts.device)
    pilot = _field(b, ih, 1.0 / float(np.prod([float(v) for v in ell])), r, "epanechnikov")
    if pilot is None:
        return None
    den = _trilinear(pilot * scale, r, b)
    mean = float(den.mean())
    ratio = torch.where(den > 0, mean / den, torch.full_like(den, math.inf)) ** (1.0 / 3.0)
    lj = torch.stack([torch.clamp(float(ell[k]) * ratio, max=5.0 * s[k]) for k in range(3)], 1).float()
    final = _field(b, (1.0 / lj.double()).float(), 1.0 / lj.double().prod(1), r, "epanechnikov")
    return None if final is None else final * scale


def exact(case, seed):
    kind, n = case["kind"], case["points"]
    if kind in ("batch", "serve") or (case["knn"] and n > 150_000):
        return None
    pts, tops = _cloud(n, seed)
    r = _regions(case, seed, tops)[0]
    if kind == "consume":
        grid = _counts(pts, r)
        v = torch.zeros(n, dtype=torch.float64, device=pts.device)
        for a in range(0, n, 1 << 23):
            p = pts[a:a + (1 << 23)]
            v[a:a + (1 << 23)] = torch.where(_inside(p, r), _trilinear(grid, r, p), v[a:a + (1 << 23)])
        return {"density": v, "selected": None, "surface": None}
    if case["bw"] == "mbe":
        return _adaptive(pts, r)
    count = n
    if case["bw"] == "per_point":
        if case["knn"]:
            h = torch.sqrt(_neighbour_h2(pts, case["knn"]).double())
        else:
            h = _lengths(pts, seed).double()
        ih = (1.0 / h).float()[:, None].expand(n, 3)
        w = 1.0 / h ** 3
    else:
        h = [float(np.float32(r.h[k])) if case["bw"] == "fixed"
             else float(np.float32(float(np.float32(r.h[0])) * (r.hi[k] - r.lo[k]))) for k in range(3)]
        ih = torch.tensor([1.0 / v for v in h], dtype=torch.float32, device=pts.device)
        w = 1.0 / (h[0] * h[1] * h[2])
    if case["set"] == "in_roi":
        inside = _inside(pts, r)
        count = int(inside.sum())
        if count == 0:
            return torch.zeros(r.n_nodes, dtype=torch.float64, device=pts.device)
        pts = pts[inside]
        if ih.dim() == 2:
            ih, w = ih[inside], w[inside]
    grid = _field(pts, ih, w, r, case["kernel"])
    return None if grid is None else grid * (_ck(case["kernel"]) * (1.0 if case["norm"] == "count" else 1.0 / count))
