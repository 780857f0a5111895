"""Workloads of the shadow-accumulation library, as its users run them.

Each case is one call (or one forward and backward step) on a synthetic
Manhattan-like city: convex footprints of 4 to 12 vertices on 40 x 27 m
parcels, 2 x 10 parcels a block, 18 m streets, lognormal heights; ground
points on a square lattice in the open space nearest the centre, in Morton
order, and facade points on wall cells of the buildings nearest it, with
their owner and outward normal.  Everything is drawn from the seed; the
cities, point sets and dates are those of the library's own benchmark and
tests in kind and size.

``exact`` gives the same results in 64 bits by brute force (every prism
against every point), where that takes seconds.
"""
import functools
import math

import numpy as np
import torch

import paper_1907_04435_amd as sa

BLOCK_W, BLOCK_D, STREET = 80.0, 270.0, 18.0
PARCEL_W, PARCEL_D = 40.0, 27.0
MAX_V = 12  # vertices of the largest footprint

# dates used by the library's benchmark: both solstices and an equinox
DATES = [(2019, 3, 20), (2019, 6, 21), (2019, 12, 21)]


def _case(name, kind, prisms, points, **kw):
    c = {"name": name, "kind": kind, "prisms": prisms, "points": points, "facade": 0.5, "pitch": 1.0, "days": 1,
         "date": 1, "lat": 40.7, "step": 1.0, "seg": 30.0, "median": 20.0}
    c.update(kw)
    return c


def listed():
    return [
        # a building site under study: one call's latency counts (64 prisms,
        # 16,384 ground points on a 4 m lattice, a working day at 5 minutes)
        _case("site_accrual", "accrual", 64, 16384, facade=0.0, pitch=4.0, step=5.0, window=True, median=60.0),
        # interactive design: eight heights change, the neighbourhood is accrued again
        _case("edit_accrual", "edit", 400, 40000, edits=8),
        # the headline: a borough's ground and facades over three days
        _case("block_accrual", "accrual", 20000, 4000000, days=3),
        # per-instant rays over a neighbourhood (ragged point count)
        _case("hood_sampled", "sampled", 400, 20011),
        # per-instant rays over a borough
        _case("block_sampled", "sampled", 20000, 1000000, days=3),
        # per-instant bit vectors kept for later queries
        _case("block_bits", "bits", 20000, 200003, days=2),
        # longest uninterrupted shadow beside the total
        _case("block_runs", "runs", 20000, 500000, days=3),
        # which building shades the points, weighted
        _case("contribution", "contribution", 5000, 300000, days=2),
        # optimising heights: minutes of a park and their gradient, knots at every minute
        _case("park_gradient", "gradient", 5000, 200000, facade=0.0, seg=1.0, date=0, median=30.0),
        # development variants compared in one call
        _case("variants", "batched", 20000, 1000000, facade=0.0, days=2, variants=32, edits=8),
        # a whole year in four season bins
        _case("year_seasons", "year", 45000, 500000, facade=0.0, days=365),
        # raster maps for exploration, 2 m texels
        _case("raster", "raster", 20000, 1000000, facade=0.0, texel=2.0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["accrual", "edit", "sampled", "bits", "runs", "sampled_runs", "contribution", "gradient",
                       "batched", "year", "graph", "raster"])
    c = _case("", kind, _log(rng, 40, 20000), _log(rng, 3000, 1000000))
    del c["name"]
    c["date"] = rng.randrange(3)
    c["lat"] = round(rng.uniform(25.0, 52.0), 3)
    c["days"] = rng.randint(1, 3)
    c["facade"] = rng.choice([0.0, 0.3, 0.5, 1.0])
    c["seg"] = rng.choice([15.0, 20.0, 30.0, 45.0, 60.0])
    c["median"] = round(rng.uniform(15.0, 40.0), 2)
    c["pitch"] = rng.choice([1.0, 1.0, 2.0, 4.0])
    if kind in ("accrual", "runs"):
        c["points"] = _log(rng, 3000, 3000000)
        c["step"] = rng.choice([1.0, 5.0])
    if kind in ("sampled", "sampled_runs", "bits"):
        c["step"] = rng.choice([1.0, 1.0, 2.0, 5.0, 10.0])
        c["points"] = _log(rng, 3000, 500000)
    if kind == "edit":
        c["edits"] = rng.randint(1, 16)
    if kind == "gradient":
        c["seg"] = rng.choice([1.0, 2.0, 5.0, 30.0])
        c["prisms"] = _log(rng, 100, 6000)
        c["points"] = _log(rng, 3000, 200000)
        c["facade"] = 0.0
        c["days"] = 1
    if kind == "batched":
        c["facade"] = 0.0
        c["variants"] = rng.randint(2, 48)
        c["edits"] = rng.randint(1, 12)
    if kind in ("year", "graph"):
        c["days"] = rng.randint(40, 365)
        c["points"] = _log(rng, 3000, 200000)
        c["facade"] = 0.0
        if kind == "graph":
            c["bound"] = rng.choice([0.5, 1.0, 3.0, 5.0])
    if kind == "raster":
        c["facade"] = 0.0
        c["days"] = 1
        c["step"] = rng.choice([1.0, 5.0])
        c["texel"] = rng.choice([1.5, 2.0, 4.0])
    return c


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _city(rng, n, median):
    """(vert_off int32, xy float32, height float32, parcel -> prism map, cols, rows)."""
    blocks = max(1, math.ceil(n / 20 * 1.08))
    cols = max(1, min(35, int(round(math.sqrt(blocks * (BLOCK_D + STREET) / (BLOCK_W + STREET) * 0.33)))))
    rows = -(-blocks // cols)
    par = np.sort(rng.choice(cols * rows * 20, size=n, replace=False))
    pc, pr = par % (cols * 2), par // (cols * 2)
    cx = (pc // 2) * (BLOCK_W + STREET) + (pc % 2) * PARCEL_W + PARCEL_W / 2
    cy = (pr // 10) * (BLOCK_D + STREET) + (pr % 10) * PARCEL_D + PARCEL_D / 2
    ax = (PARCEL_W / 2 - 1.0) * rng.uniform(0.6, 1.0, n)
    ay = (PARCEL_D / 2 - 1.0) * rng.uniform(0.6, 1.0, n)
    m = rng.integers(4, MAX_V + 1, n)
    ang = np.full((n, MAX_V), np.inf)
    todo = np.arange(n)
    while len(todo):  # sorted angles, no two closer than pi / 2m
        a = np.where(np.arange(MAX_V) < m[todo, None], rng.uniform(0, 2 * np.pi, (len(todo), MAX_V)), np.inf)
        a.sort(axis=1)
        ext = np.concatenate([a, np.full((len(todo), 1), np.inf)], 1)
        ext[np.arange(len(todo)), m[todo]] = a[:, 0] + 2 * np.pi
        gaps = np.where(np.arange(MAX_V) < m[todo, None], ext[:, 1:], np.inf) - np.where(np.isfinite(a), a, 0.0)
        ok = gaps.min(1) >= np.pi / (2 * m[todo])
        ang[todo[ok]] = a[ok]
        todo = todo[~ok]
    use = np.arange(MAX_V) < m[:, None]
    an = np.where(use, ang, 0.0)
    xy = np.stack([cx[:, None] + ax[:, None] * np.cos(an), cy[:, None] + ay[:, None] * np.sin(an)], -1)
    xy = xy[use].astype(np.float32)
    off = np.concatenate([[0], np.cumsum(m)]).astype(np.int32)
    h = np.clip(median * np.exp(rng.standard_normal(n)), 3.0, 400.0).astype(np.float32)
    of_parcel = np.full(cols * rows * 20, -1, np.int64)
    of_parcel[par] = np.arange(n)
    return off, xy, h, of_parcel, cols, rows


def _padded(off, xy):
    """Footprints as [n, MAX_V, 2] float64 on the GPU, the last vertex repeated."""
    m = np.diff(off)
    at = off[:-1, None] + np.minimum(np.arange(MAX_V), m[:, None] - 1)
    return torch.from_numpy(xy.astype(np.float64)[at]).cuda()


def _ground(city, poly, n, pitch):
    """The n open lattice points nearest the centre (Chebyshev), Morton order."""
    _, _, _, of_parcel, cols, rows = city
    ex, ey = cols * (BLOCK_W + STREET) - STREET, rows * (BLOCK_D + STREET) - STREET
    # a square about the centre with room for the footprints; a small city's surroundings count too
    r = (math.sqrt(n / 0.4) / 2 + 8) * pitch
    x0, x1, y0, y1 = ex / 2 - r, ex / 2 + r, ey / 2 - r, ey / 2 + r
    nx, ny = int((x1 - x0) / pitch) + 1, int((y1 - y0) / pitch) + 1
    cells = torch.arange(nx * ny, device="cuda")
    gx = x0 + (cells % nx).double() * pitch + 0.5
    gy = y0 + torch.div(cells, nx, rounding_mode="floor").double() * pitch + 0.5
    cheb = torch.maximum((gx - ex / 2).abs(), (gy - ey / 2).abs())
    near = torch.argsort(cheb, stable=True)
    gx, gy = gx[near], gy[near]
    bc, br = torch.floor(gx / (BLOCK_W + STREET)), torch.floor(gy / (BLOCK_D + STREET))
    lx, ly = gx - bc * (BLOCK_W + STREET), gy - br * (BLOCK_D + STREET)
    on = (gx >= 0) & (gx < ex) & (gy >= 0) & (gy < ey) & (lx < BLOCK_W) & (ly < BLOCK_D)
    p = (br * 10 + torch.floor(ly / PARCEL_D).clamp(max=9)) * (cols * 2) + bc * 2 + torch.floor(lx / PARCEL_W).clamp(max=1)
    b = torch.from_numpy(of_parcel).cuda()[torch.where(on, p, 0.0).long()]
    on &= b >= 0
    inside = on.clone()
    q = poly[b.clamp(min=0)]
    for k in range(MAX_V):
        e = q[:, (k + 1) % MAX_V] - q[:, k]
        ln = e.norm(dim=1).clamp(min=1e-9)
        inside &= ((gx - q[:, k, 0]) * e[:, 1] - (gy - q[:, k, 1]) * e[:, 0]) / ln <= 0.05
    gx, gy = gx[~inside][:n].float(), gy[~inside][:n].float()
    ix, iy = torch.floor(gx - gx.min()).long(), torch.floor(gy - gy.min()).long()
    code = torch.zeros_like(ix)
    for k in range(16):
        code |= ((ix >> k) & 1) << (2 * k) | ((iy >> k) & 1) << (2 * k + 1)
    o = torch.argsort(code, stable=True)
    return gx[o], gy[o]


def _facade(city, n):
    """1 m wall cells of the buildings nearest the centre: x, y, z, nx, ny, owner."""
    off, xy, h, _, cols, rows = city
    c = np.array([(cols * (BLOCK_W + STREET) - STREET) / 2, (rows * (BLOCK_D + STREET) - STREET) / 2])
    b_of = np.repeat(np.arange(len(h)), np.diff(off))
    v = xy.astype(np.float64)
    nxt = np.arange(len(v)) + 1
    nxt[off[1:] - 1] = off[:-1]
    e = v[nxt] - v
    ln = np.hypot(e[:, 0], e[:, 1])
    cen = np.add.reduceat(v, off[:-1], axis=0) / np.diff(off)[:, None]
    rank = np.argsort(np.argsort(np.hypot(*(cen - c).T), kind="stable"), kind="stable")
    ed = np.argsort(rank[b_of], kind="stable")
    ncol, nrow = np.floor(ln[ed]).astype(np.int64), np.floor(h[b_of[ed]]).astype(np.int64)
    cells = np.cumsum(ncol * nrow)
    last = int(np.searchsorted(cells, n)) + 1
    ed, ncol, nrow = (torch.from_numpy(a[:last]).cuda() for a in (ed, ncol, nrow))
    cnt = ncol * nrow
    which = torch.repeat_interleave(torch.arange(len(ed), device="cuda"), cnt)[:n]
    i = torch.arange(len(which), device="cuda") - (torch.cumsum(cnt, 0) - cnt)[which]
    t = torch.div(i, nrow[which], rounding_mode="floor").double() + 0.5
    z = (i % nrow[which]).float() + 0.5
    E = ed[which]
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()[E]  # noqa: E731
    ux, uy = g(e[:, 0] / ln), g(e[:, 1] / ln)
    return ((g(v[:, 0]) + t * ux).float(), (g(v[:, 1]) + t * uy).float(), z, uy.float(), (-ux).float(),
            g(b_of.astype(np.int32)))


def _sun(case):
    """The library's sun path: instants, weights and knots of the case's days."""
    lat, lon, tz, step, seg = case["lat"], -74.0, -5.0, case["step"], case["seg"]
    if case["kind"] in ("year", "graph"):
        sp = sa.sa_sunpath(lat, lon, tz, 2019, 1, 1, case["days"], -1.0, -1.0, step, seg)
        sp.day_bin = (np.arange(case["days"]) // 92).astype(np.int32)
        return sp
    t0, t1 = (480.0, 1080.0) if case.get("window") else (-1.0, -1.0)
    return sa.concat_paths([sa.sa_sunpath(lat, lon, tz, *DATES[(case["date"] + k) % 3], 1, t0, t1, step, seg)
                            for k in range(case["days"])])


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    city = _city(rng, case["prisms"], case["median"])
    off, xy, h = city[:3]
    n = case["points"]
    n_f = int(n * case["facade"])
    parts = []
    if n > n_f:
        gx, gy = _ground(city, _padded(off, xy), n - n_f, case["pitch"])
        zero = torch.zeros_like(gx)
        parts.append((gx, gy, zero, zero, zero, torch.full(gx.shape, -1, dtype=torch.int32, device="cuda")))
    if n_f:
        parts.append(_facade(city, n_f))
    pts = [torch.cat(a).contiguous() for a in zip(*parts)]
    got = {"off": off, "xy": xy, "h": h, "pts": pts, "sun": _sun(case)}
    n = len(pts[0])
    if case["kind"] == "edit":
        got["ids"] = np.sort(rng.choice(len(h), min(len(h), case["edits"]), replace=False)).astype(np.int32)
        got["new_h"] = rng.uniform(20.0, 200.0, len(got["ids"])).astype(np.float32)
    if case["kind"] == "contribution":
        got["weight"] = torch.from_numpy(rng.uniform(0.25, 2.0, n).astype(np.float32)).cuda()
    if case["kind"] == "batched":
        V, k = case["variants"], min(len(h), case["edits"])
        cut = np.sort(rng.integers(0, n + 1, V - 1))
        got["var_off"] = np.concatenate([[0], cut, [n]]).astype(np.int64)
        got["ids"] = np.stack([np.sort(rng.choice(len(h), k, replace=False)) for _ in range(V)]).astype(np.int32)
        got["new_h"] = rng.uniform(50.0, 400.0, (V, k)).astype(np.float32)
    if case["kind"] == "gradient":
        got["dl"] = torch.from_numpy(rng.uniform(0.5, 1.5, (1, n)).astype(np.float32)).cuda()
    return got


@functools.lru_cache(maxsize=1)
def _context():
    """A program opens the device once and keeps the handle."""
    return sa.Context(0)


def prepare(case, seed):
    d = _inputs(case, seed)
    ctx, kind = _context(), case["kind"]
    s = {"kind": kind, "ctx": ctx, "scene": sa.Scene(ctx, d["off"], d["xy"], d["h"]),
         "path": sa.Path(ctx, d["sun"], case.get("bound"))}
    x, y, z, nx, ny, own = d["pts"]
    s["pts"] = sa.DevicePoints(x, y, z) if kind == "raster" else sa.DevicePoints(x, y, z, nx, ny, own)
    B, n = s["path"].n_bins, s["pts"].n
    out = lambda t, *shape: torch.empty(shape, dtype=t, device="cuda")  # noqa: E731
    if kind in ("accrual", "batched"):
        s["out"] = [out(torch.int32, B, n), out(torch.float32, B, n)]
    if kind == "sampled_runs":
        s["out"] = [out(torch.int32, B, n), out(torch.float32, B, n), out(torch.float32, B, n)]
    if kind in ("year", "graph"):
        s["out"] = [out(torch.float32, B, n)]
    if kind == "edit":
        s["ids"], s["new_h"] = d["ids"], d["new_h"]
    if kind == "contribution":
        s["weight"] = d["weight"]
    if kind == "batched":
        s["ids"], s["new_h"], s["var_off"] = (torch.from_numpy(d[k]).cuda() for k in ("ids", "new_h", "var_off"))
    if kind == "gradient":
        s["fn"] = sa.shadow_minutes_fn()
        s["heights"] = torch.from_numpy(d["h"]).cuda().requires_grad_(True)
        s["dl"] = d["dl"]
    if kind == "raster":
        s["texel"] = case["texel"]
    torch.cuda.synchronize()
    return s


def run(s):
    kind, ctx, scene, pts, path = s["kind"], s["ctx"], s["scene"], s["pts"], s["path"]
    if kind == "accrual":
        sa.sa_accumulate(ctx, scene, pts, path, sa.SA_ACCRUAL, *s["out"])
        return s["out"]
    if kind in ("year", "graph"):
        sa.sa_accumulate(ctx, scene, pts, path, sa.SA_ACCRUAL, None, s["out"][0], out_scale=1.0 / 60.0)
        return s["out"]
    if kind == "edit":
        scene.set_heights(s["ids"], s["new_h"])
        return sa.accumulate(ctx, scene, pts, path, sa.SA_ACCRUAL)[:2]
    if kind == "sampled":
        return sa.accumulate(ctx, scene, pts, path, sa.SA_SAMPLED)[:2]
    if kind == "bits":
        return sa.accumulate(ctx, scene, pts, path, sa.SA_SAMPLED, want_bits=True)
    if kind == "sampled_runs":
        sa.sa_accumulate(ctx, scene, pts, path, sa.SA_SAMPLED, s["out"][0], s["out"][1], longest=s["out"][2])
        return s["out"]
    if kind == "runs":
        return sa.continuous_shadow(ctx, scene, pts, path, sa.SA_ACCRUAL)
    if kind == "contribution":
        return sa.building_contribution(ctx, scene, pts, path, s["weight"])
    if kind == "gradient":
        minutes = s["fn"].apply(s["heights"], ctx, scene, pts, path)
        (grad,) = torch.autograd.grad(minutes, s["heights"], s["dl"])
        return minutes.detach(), grad
    if kind == "batched":
        sa.sa_accumulate_batched(ctx, scene, s["ids"], s["new_h"], pts, s["var_off"], path, *s["out"])
        return s["out"]
    if kind == "raster":
        return sa.sam_accumulate(ctx, scene, pts, path, s["texel"])
    raise ValueError(kind)


def work(case):
    """Bytes: points, footprints, heights and sun path read once, outputs
    written once.  Operations: one prism decided per point and segment (40 and
    10 an edge) or per point and instant (6 and 8 an edge; 4 for a raster
    lookup), 8 edges a prism; the gradient's step decides them twice."""
    kind, n, b = case["kind"], case["points"], case["prisms"]
    year = kind in ("year", "graph")
    bins = min(4, -(-case["days"] // 92)) if year else case["days"]
    span = 600.0 if case.get("window") else 730.0
    inst = case["days"] * span / case["step"]
    segs = case["days"] * span / case["seg"]
    out = n * bins * {"bits": 8, "sampled_runs": 12, "year": 4, "graph": 4, "contribution": 0, "gradient": 8}.get(kind, 8)
    if kind == "bits":
        out += n * inst / 8
    if kind == "contribution":
        out += 8 * b * bins
    if kind == "gradient":
        out += 4 * b
    data = n * (12 if kind == "raster" else 24) + b * (8 * 8 + 8) + inst * 32 + segs * 24 + out
    if kind in ("sampled", "bits", "sampled_runs"):
        ops = n * inst * (6 + 8 * 8)
    elif kind == "raster":
        ops = n * inst * 4
    else:
        ops = n * segs * (40 + 10 * 8) * (2 if kind == "gradient" else 1)
    return {"bytes": float(data), "flops": float(ops)}


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------
def _windows(sun):
    """Great-circle segments: (day, bin, dt, theta, e1, e2)."""
    for d in range(len(sun.day_bin)):
        k0, k1 = sun.day_knot_off[d], sun.day_knot_off[d + 1]
        for k in range(k0, k1 - 1):
            a, b = sun.knot_dir[k], sun.knot_dir[k + 1]
            e2 = b - np.dot(a, b) * a
            th = math.atan2(np.linalg.norm(np.cross(a, b)), float(np.dot(a, b)))
            yield d, int(sun.day_bin[d]), sun.knot_t[k + 1] - sun.knot_t[k], th, a, e2 / np.linalg.norm(e2)


def _clip_to(lo, hi, th):
    """[lo, hi] (any branch of the angle, shorter than a half turn or one) within [0, th]; empty: a > b."""
    turn = 2 * math.pi * torch.round(((lo + hi) / 2 - th / 2) / (2 * math.pi))
    return (lo - turn).clamp(min=0.0), (hi - turn).clamp(max=th)


def _pairs(P, poly, H, th, e1, e2):
    """Occluded angles [a, b] of every (point, prism), and a last column for
    walls facing away from the sun; a > b where there is none."""
    px, py, pz, nx, ny, own = P
    n = np.cross(e1, e2)
    wx, wy = poly[None, :, :, 0] - px[:, None, None], poly[None, :, :, 1] - py[:, None, None]
    z = -(n[0] * wx + n[1] * wy) / n[2]
    h = (H[None, :] - pz[:, None])[:, :, None]
    in_plane = lambda x, y, t: (e1[0] * x + e1[1] * y + e1[2] * t, e2[0] * x + e2[1] * y + e2[2] * t)  # noqa: E731
    ex, ey, ez = (torch.roll(a, -1, 2) - a for a in (wx, wy, z))
    inside = (wx * (wy + ey) - wy * (wx + ex) >= 0).all(2)
    below = z <= h
    cross = below != torch.roll(below, -1, 2)
    t = torch.where(cross, (h - z) / torch.where(cross, ez, 1.0), 0.0)
    u, v = in_plane(wx, wy, z)
    cu, cv = in_plane(wx + t * ex, wy + t * ey, h.expand_as(z))
    u, v, ok = torch.cat([u, cu], 2), torch.cat([v, cv], 2), torch.cat([below, cross], 2)
    mu, mv = torch.where(ok, u, 0.0).sum(2, keepdim=True).detach(), torch.where(ok, v, 0.0).sum(2, keepdim=True).detach()
    su, sv = torch.where(ok, u, mu + 1e-300), torch.where(ok, v, mv)
    rel = torch.atan2(mu * sv - mv * su, mu * su + mv * sv)
    ref = torch.atan2(mv, mu)[:, :, 0]
    some = ok.any(2)
    lo = torch.where(ok, rel, math.inf).amin(2)
    hi = torch.where(ok, rel, -math.inf).amax(2)
    a, b = _clip_to(torch.where(some, ref + lo, 0.0), torch.where(some, ref + hi, 0.0), th)
    over = inside & (h[:, :, 0] >= 0)
    a, b = torch.where(inside, 0.0, a), torch.where(inside, th, b)
    none = (inside & ~over) | (~inside & ~some) | (torch.arange(len(H), device=H.device)[None] == own[:, None]) | (b <= a)
    f = torch.atan2(ny * e2[1] + nx * e2[0], ny * e1[1] + nx * e1[0])  # the wall's normal in the plane
    fa, fb = _clip_to(f + math.pi / 2, f + 3 * math.pi / 2, th)
    front = (own < 0) | (fb <= fa)
    a = torch.cat([torch.where(none, 9.0, a), torch.where(front, 9.0, fa)[:, None]], 1)
    b = torch.cat([torch.where(none, -9.0, b), torch.where(front, -9.0, fb)[:, None]], 1)
    return a, b


def _union(a, b):
    """Sorted members: starts and ends of what each adds to the set before it (end <= start: nothing)."""
    a, o = a.sort(1)
    b = b.gather(1, o)
    top = torch.cat([torch.full_like(b[:, :1], -9.0), b.cummax(1).values[:, :-1]], 1)
    return torch.maximum(a, top), b, top


def _chunks(n, b, most=24_000_000):
    step = max(1, int(most // (b * 2 * MAX_V)))
    return [(i, min(n, i + step)) for i in range(0, n, step)]


def _points64(d):
    return [a.double() for a in d["pts"][:5]] + [d["pts"][5].long()]


def _accrue(d, H, P, want):
    """Minutes [bins, n] (and longest), or contributions [bins, prisms]."""
    poly, sun = _padded(d["off"], d["xy"]), d["sun"]
    bins, n, nb = int(sun.day_bin.max()) + 1, len(P[0]), len(H)
    minutes = torch.zeros((bins, n), dtype=torch.float64, device="cuda")
    longest = torch.zeros_like(minutes)
    contrib = torch.zeros((bins, nb), dtype=torch.float64, device="cuda")
    for i0, i1 in _chunks(n, nb):
        Q = [a[i0:i1] for a in P]
        run, day = torch.zeros(i1 - i0, dtype=torch.float64, device="cuda"), -1
        for dd, bin_, dt, th, e1, e2 in _windows(sun):
            a, b = _pairs(Q, poly, H, th, e1, e2)
            if want == "contribution":
                part = (b - a).clamp(min=0.0) * d["weight"][i0:i1, None].double() * (dt / th)
                contrib[bin_] += part[:, :nb].sum(0)
                facade = Q[5] >= 0
                contrib[bin_].index_add_(0, Q[5][facade], part[facade, nb])
                continue
            lo, hi, top = _union(a, b)
            minutes[bin_, i0:i1] += (hi - lo).clamp(min=0.0).sum(1) * (dt / th)
            if want != "runs":
                continue
            if dd != day:
                run, day = torch.zeros_like(run), dd
            best = longest[bin_, i0:i1]
            reach = torch.zeros_like(run)  # the set so far ends here; run counts up to it
            for k in range(int((hi > lo).sum(1).max()) + int((hi <= lo).sum(1).max()) if len(hi) else 0):
                add = hi[:, k] > lo[:, k]
                if not bool(add.any()):
                    if bool((lo[:, k] >= 9.0).all()):
                        break
                    continue
                joins = lo[:, k] <= reach
                run = torch.where(add, torch.where(joins, run, 0.0) + (hi[:, k] - lo[:, k]) * (dt / th), run)
                reach = torch.where(add, hi[:, k], reach)
                best = torch.where(add, torch.maximum(best, run), best)
            longest[bin_, i0:i1] = best
            run = torch.where(reach >= th, run, 0.0)
    return contrib if want == "contribution" else (minutes, longest)


def _rays(d, H, P):
    """Sampled minutes and longest runs: every ray against every prism."""
    poly, sun = _padded(d["off"], d["xy"]), d["sun"]
    bins, n, nb = int(sun.day_bin.max()) + 1, len(P[0]), len(H)
    minutes = torch.zeros((bins, n), dtype=torch.float64, device="cuda")
    longest = torch.zeros_like(minutes)
    e = torch.roll(poly, -1, 1) - poly
    flat = (e == 0).all(2)  # repeated vertices
    for i0, i1 in _chunks(n, nb, 40_000_000):
        px, py, pz, nx, ny, own = (a[i0:i1] for a in P)
        num = e[None, :, :, 1] * (poly[None, :, :, 0] - px[:, None, None]) - e[None, :, :, 0] * (poly[None, :, :, 1] - py[:, None, None])
        mine = torch.arange(nb, device="cuda")[None] == own[:, None]
        for dd in range(len(sun.day_bin)):
            bin_ = int(sun.day_bin[dd])
            run = torch.zeros(i1 - i0, dtype=torch.float64, device="cuda")
            for k in range(sun.day_sample_off[dd], sun.day_sample_off[dd + 1]):
                dx, dy, dz = (float(v) for v in np.asarray(sun.dir).reshape(-1, 3)[k])
                den = e[:, :, 1] * dx - e[:, :, 0] * dy
                s = num / torch.where(den == 0, 1.0, den)
                s_out = torch.where(den > 0, s, math.inf).amin(2)
                s_in = torch.where(den < 0, s, 0.0).amax(2).clamp(min=0.0)
                miss = ((den == 0) & ~flat & (num < 0)).any(2)
                hit = (s_out >= s_in) & (pz[:, None] + s_in * dz <= H[None]) & ~miss & ~mine
                sh = hit.any(1) | ((own >= 0) & (nx * dx + ny * dy <= 0))
                w = float(sun.weight[k])
                minutes[bin_, i0:i1] += w * sh
                run = torch.where(sh, run + w, 0.0)
                longest[bin_, i0:i1] = torch.maximum(longest[bin_, i0:i1], run)
    return minutes, longest


def exact(case, seed):
    kind, n, b = case["kind"], case["points"], case["prisms"]
    span = case["days"] * (600.0 if case.get("window") else 730.0)
    rays = kind in ("sampled", "bits", "sampled_runs")
    # a raster count is decided by texels and quantised depths: it has no value of its own
    pairs = n * b * span / (case["step"] if rays else case["seg"])
    if kind in ("raster", "graph", "year") or pairs > {"gradient": 2e8}.get(kind, 6e9 if rays else 1.5e9):
        return None
    d = _inputs(case, seed)
    H, P = torch.from_numpy(d["h"]).cuda().double(), _points64(d)
    if rays:
        minutes, longest = _rays(d, H, P)
        return [None, minutes, longest] if kind == "sampled_runs" else [None, minutes] + [None] * (kind == "bits")
    if kind == "edit":
        H[torch.from_numpy(d["ids"]).long().cuda()] = torch.from_numpy(d["new_h"]).double().cuda()
    if kind in ("accrual", "edit"):
        return [None, _accrue(d, H, P, "minutes")[0]]
    if kind == "runs":
        return list(_accrue(d, H, P, "runs"))
    if kind == "contribution":
        return _accrue(d, H, P, "contribution")
    if kind == "batched":
        parts = []
        for v in range(case["variants"]):
            Hv = H.clone()
            Hv[torch.from_numpy(d["ids"][v]).long().cuda()] = torch.from_numpy(d["new_h"][v]).double().cuda()
            i0, i1 = d["var_off"][v], d["var_off"][v + 1]
            if i1 > i0:
                parts.append(_accrue(d, Hv, [a[i0:i1] for a in P], "minutes")[0])
        return [None, torch.cat(parts, 1)]
    # the gradient of the union's measure, by differentiating the 64-bit minutes
    grad, minutes = torch.zeros_like(H), []
    for i0, i1 in _chunks(n, b, 3_000_000):
        Q = [a[i0:i1] for a in P]
        got = torch.zeros((1, i1 - i0), dtype=torch.float64, device="cuda")
        for _, _, dt, th, e1, e2 in _windows(d["sun"]):
            Hv = H.clone().requires_grad_(True)
            a, bb = _pairs(Q, _padded(d["off"], d["xy"]), Hv, th, e1, e2)
            lo, hi, _ = _union(a, bb)
            m = (hi - lo).clamp(min=0.0).sum(1) * (dt / th)
            grad += torch.autograd.grad((m * d["dl"][0, i0:i1]).sum(), Hv)[0]
            got[0] += m.detach()
        minutes.append(got)
    return [torch.cat(minutes, 1), grad]
