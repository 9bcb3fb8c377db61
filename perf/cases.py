"""Timed cases of the distance-bounded aggregation join: what a program that
uses this library does with it, from the smallest calls to the largest.

A case is a dict of plain values.  Its "kind" is the call that it stands for:

* step         build the approximation of a polygon set and answer COUNT and
               SUM of a batch of points from it (ad-hoc polygons, or a new
               distance bound);
* probe        a standing handle and a new batch of points;
* range        the result range [alpha - beta, alpha] over a batch of points;
* viewports    map queries: per viewport a clip-window build at one pixel's
               distance bound, then all of them answered in one batch over the
               resident, bucketed points;
* runs         points against a standing quadtree (Hilbert run) handle of many
               polygons;
* partitioned  the same through the call that first partitions the points;
* pindex_build pre-aggregation of a new batch of points, and the standing
               query answered from it;
* pindex_query new polygons against a standing point index;
* join         pairs of polygons of two sets whose approximations meet.

All inputs are synthetic and made from the seed alone: points are uniform or a
mixture of 50 Gaussians (a city's pickups), values cents, polygons random
stars or a partition of the box with jittered edges (census blocks).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2010_12548_amd as sba

DEV = torch.device("cuda" if torch.cuda.is_available() else "cpu")
TINY_BOX = 65_536     # coordinates of the star workload
CITY_BOX = 4_000_000  # 40 km at 1 cm per unit

# Edge vertices per shared side: neighbourhoods (hundreds of polygons) are
# finely drawn, census blocks (tens of thousands) have 32-332 vertices each.
COARSE, FINE = (10, 200), (8, 83)


def listed():
    return [
        # the smallest whole query: 16 overlapping polygons over a million
        # uniform points; the build's launches and read-backs weigh most
        {"name": "step_stars", "kind": "step", "stars": 16, "polys": 0, "eps": 64,
         "points": 1_000_000, "values": True},
        # the headline workload: 260 neighbourhoods, 10 m, 1e8 pickups
        {"name": "step_city_10m", "kind": "step", "stars": 0, "polys": 260, "eps": 1000,
         "points": 100_000_000, "values": True},
        # the finest bound in use (1 m): a build of a hundred times the cells
        {"name": "step_city_1m", "kind": "step", "stars": 0, "polys": 260, "eps": 100,
         "points": 30_000_001, "values": True},
        # the smallest call: a trickle of points against a standing handle
        {"name": "probe_small", "kind": "probe", "polys": 260, "eps": 1000, "points": 20_001,
         "values": True},
        # COUNT only (no values are read), 100 m, an odd number of points
        {"name": "probe_count_100m", "kind": "probe", "polys": 260, "eps": 10_000,
         "points": 33_333_333, "values": False},
        # exact answers bounded from both sides
        {"name": "range_city_10m", "kind": "range", "polys": 260, "eps": 1000,
         "points": 50_000_000, "values": True},
        # a screen of map queries at mixed zoom levels
        {"name": "viewports_16", "kind": "viewports", "polys": 4000, "queries": 16,
         "points": 50_000_000},
        # census blocks at 1 m, points as they arrive (no spatial order)
        {"name": "runs_blocks_1m", "kind": "runs", "polys": 40_000, "eps": 100,
         "points": 20_000_000, "values": True, "search": "learned", "ordered": False},
        # the same polygons, a large batch through the partitioning call
        {"name": "partitioned_blocks_1m", "kind": "partitioned", "polys": 40_000, "eps": 100,
         "points": 100_000_000, "values": True, "search": "binary"},
        # pre-aggregation of a day's points
        {"name": "pindex_build_1m", "kind": "pindex_build", "polys": 260, "eps": 100,
         "points": 50_000_000, "values": True},
        # census blocks answered from pre-aggregated points
        {"name": "pindex_query_blocks_1m", "kind": "pindex_query", "polys": 40_000, "eps": 100,
         "points": 20_000_000, "values": True, "search": "learned"},
        # census blocks against neighbourhoods
        {"name": "join_blocks_city_1m", "kind": "join", "polys": 40_000, "polys2": 260,
         "eps": 100},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))


def draw(rng):
    kind = rng.choice(["step", "step", "probe", "probe", "range", "viewports", "runs",
                       "partitioned", "pindex_build", "pindex_query", "join"])
    values = rng.random() < 0.7
    if kind == "step":
        if rng.random() < 0.3:
            return {"kind": kind, "stars": _log_int(rng, 12, 64), "polys": 0,
                    "eps": _log_int(rng, 64, 600), "points": _log_int(rng, 50_000, 10_000_000),
                    "values": values}
        return {"kind": kind, "stars": 0, "polys": _log_int(rng, 40, 2000),
                "eps": _log_int(rng, 100, 12_000), "points": _log_int(rng, 100_000, 60_000_000),
                "values": values}
    if kind == "probe":
        return {"kind": kind, "polys": _log_int(rng, 40, 2000), "eps": _log_int(rng, 100, 12_000),
                "points": _log_int(rng, 2_000, 90_000_000), "values": values}
    if kind == "range":
        return {"kind": kind, "polys": _log_int(rng, 60, 600), "eps": _log_int(rng, 300, 12_000),
                "points": _log_int(rng, 1_000_000, 60_000_000), "values": values}
    if kind == "viewports":
        return {"kind": kind, "polys": rng.choice([260, 4000]), "queries": rng.randint(1, 16),
                "points": _log_int(rng, 2_000_000, 50_000_000)}
    if kind == "runs":
        return {"kind": kind, "polys": _log_int(rng, 5_000, 40_000), "eps": _log_int(rng, 100, 400),
                "points": _log_int(rng, 200_000, 20_000_000), "values": values,
                "search": rng.choice(["learned", "binary"]), "ordered": rng.random() < 0.4}
    if kind == "partitioned":
        return {"kind": kind, "polys": _log_int(rng, 5_000, 40_000),
                "eps": _log_int(rng, 100, 400), "points": _log_int(rng, 1_000_000, 60_000_000),
                "values": values, "search": rng.choice(["learned", "binary"])}
    if kind == "pindex_build":
        return {"kind": kind, "polys": 260, "eps": _log_int(rng, 100, 2_000),
                "points": _log_int(rng, 500_000, 50_000_000), "values": values}
    if kind == "pindex_query":
        return {"kind": kind, "polys": _log_int(rng, 100, 30_000), "eps": _log_int(rng, 100, 1_000),
                "points": _log_int(rng, 1_000_000, 20_000_000), "values": values,
                "search": rng.choice(["learned", "binary"])}
    return {"kind": "join", "polys": _log_int(rng, 500, 30_000), "polys2": _log_int(rng, 40, 600),
            "eps": _log_int(rng, 100, 1_000)}


# ---------------------------------------------------------------- inputs

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + stream)
    return g


def _rand(g, *shape):
    return torch.rand(shape, generator=g, device=DEV, dtype=torch.float32)


def _uniform_points(n, box, g):
    return torch.randint(0, box, (2 * n,), generator=g, device=DEV, dtype=torch.int32)


def _mixture_points(n, box, g, k=50):
    """Gaussian mixture in [0, box)^2 (sigma 0.5-7.5 % of the box), samples
    outside drawn again; int32 [2n], in no order."""
    centres = _rand(g, k, 2) * box
    sigma = (0.005 + 0.07 * _rand(g, k)) * box
    w = torch.cumsum(0.5 + _rand(g, k), 0)
    w = w / w[-1]

    def sample(m):
        c = torch.bucketize(_rand(g, m), w).clamp_(max=k - 1)
        p = torch.randn((m, 2), generator=g, device=DEV, dtype=torch.float32)
        return p.mul_(sigma[c].unsqueeze(1)).add_(centres[c])

    def outside(p):
        return ((p < 0) | (p >= box)).any(1)

    p = sample(n)
    for _ in range(6):
        bad = torch.nonzero(outside(p)).squeeze(1)
        if bad.numel() == 0:
            break
        p[bad] = sample(bad.numel())
    return p.floor_().clamp_(0, box - 1).to(torch.int32).reshape(-1)


def _cents(n, g):
    """Lognormal(7, 0.8) cents, 1 .. 1e7."""
    z = torch.randn((n,), generator=g, device=DEV, dtype=torch.float32)
    return z.mul_(0.8).add_(7.0).exp_().add_(0.5).floor_().clamp_(1, 1e7).to(torch.int64)


def _stars(n, box, g, verts=32):
    """Random star polygons, radius 3-18 % of the box, overlaps allowed."""
    c = _rand(g, n, 1, 2) * box
    ang = torch.sort(_rand(g, n, verts) * (2 * math.pi), dim=1).values
    r = (0.03 + 0.15 * _rand(g, n, verts)) * box
    v = c + torch.stack((r * torch.cos(ang), r * torch.sin(ang)), 2)
    xy = torch.floor(v + 0.5).to(torch.int32).reshape(-1)
    ring = torch.arange(n + 1, dtype=torch.int32, device=DEV)
    return ring, torch.arange(n + 1, dtype=torch.int64, device=DEV) * verts, xy


def _partition(n, box, g, edge_verts):
    """n cells of a jittered lattice over the box; every side shared by two
    cells is one polyline of edge_verts interior vertices that both use."""
    nx = max(1, int(math.ceil(math.sqrt(n))))
    ny = max(1, -(-n // nx))
    cx, cy = box / nx, box / ny
    iy, ix = torch.meshgrid(torch.arange(ny + 1, device=DEV), torch.arange(nx + 1, device=DEV),
                            indexing="ij")
    inx = ((ix > 0) & (ix < nx)).double()
    iny = ((iy > 0) & (iy < ny)).double()
    px = ix.double() * cx + inx * (_rand(g, ny + 1, nx + 1).double() - 0.5) * 0.4 * cx
    py = iy.double() * cy + iny * (_rand(g, ny + 1, nx + 1).double() - 0.5) * 0.4 * cy
    corner = torch.stack((px, py), 2).reshape(-1, 2)
    node = (iy * (nx + 1) + ix)
    # sides: horizontal (ny+1) x nx from (x, y) to (x+1, y), then vertical ny x (nx+1)
    ha, hb = node[:, :-1].reshape(-1), node[:, 1:].reshape(-1)
    va, vb = node[:-1, :].reshape(-1), node[1:, :].reshape(-1)
    a, b = torch.cat((ha, va)), torch.cat((hb, vb))
    rows = torch.arange(ny + 1, device=DEV).repeat_interleave(nx)
    cols = torch.arange(nx + 1, device=DEV).repeat(ny)
    inner = torch.cat(((rows > 0) & (rows < ny), (cols > 0) & (cols < nx)))
    m = torch.randint(edge_verts[0], edge_verts[1] + 1, (a.numel(),), generator=g, device=DEV)
    m = torch.where(inner, m, torch.zeros_like(m))
    off = torch.cat((torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(m, 0)))
    e = torch.repeat_interleave(torch.arange(a.numel(), device=DEV), m)
    i = torch.arange(e.numel(), device=DEV) - off[e]
    me = m[e].double()
    t = (i.double() + 0.2 + 0.6 * _rand(g, e.numel()).double()) / me
    A, B = corner[a[e]], corner[b[e]]
    d = B - A
    cap = torch.minimum(0.15 * torch.minimum(t, 1 - t), 0.4 / me)
    u = (2 * _rand(g, e.numel()).double() - 1) * cap
    q = A + t.unsqueeze(1) * d + u.unsqueeze(1) * torch.stack((-d[:, 1], d[:, 0]), 1)
    # every cell: bottom, right, top reversed, left reversed; each side opens with its corner
    k = torch.arange(n, device=DEV)
    r, c = k // nx, k % nx
    nh = (ny + 1) * nx
    side = torch.stack((r * nx + c, nh + r * (nx + 1) + c + 1, (r + 1) * nx + c,
                        nh + r * (nx + 1) + c), 1).reshape(-1)
    back = torch.tensor([False, False, True, True], device=DEV).repeat(n)
    first = torch.where(back, b[side], a[side])
    length = 1 + m[side]
    soff = torch.cat((torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(length, 0)))
    s = torch.repeat_interleave(torch.arange(side.numel(), device=DEV), length)
    j = torch.arange(s.numel(), device=DEV) - soff[s]
    es = side[s]
    vert = torch.where(back[s], off[es + 1] - j, off[es] + j - 1)
    pool = torch.cat((q, corner))
    xy = pool[torch.where(j == 0, q.shape[0] + first[s], vert)]
    ring = torch.arange(n + 1, dtype=torch.int32, device=DEV)
    return ring, soff[::4].contiguous(), torch.floor(xy + 0.5).to(torch.int32).reshape(-1)


def _city(n, g):
    return _partition(n, CITY_BOX, g, COARSE if n < 1000 else FINE)


class _Polys:
    """ring_off / vert_off / xy, as the library's helpers take a polygon set."""

    def __init__(self, t):
        self.ring_off, self.vert_off, self.xy = t


def _zoom(k):
    """Zoom level above 10 of query k: 14, 18, 13, 17, 12, 16, 11, 15, 10, ..."""
    return (4 + 4 * k) % 9


def _viewports(case, seed):
    """Queries at zoom 10-18: a square of 40 km * 40^(-(z-10)/8), eps one
    pixel, COUNT and SUM in turn; the zoom levels in turn, so that a screen
    has both the whole city and single streets."""
    r = np.random.default_rng([int(seed), 77])
    out = []
    for k in range(case["queries"]):
        z = 10 + _zoom(k)
        side = int(CITY_BOX * 40.0 ** (-(z - 10) / 8.0) * r.uniform(0.8, 1.0))
        x = int(r.integers(0, CITY_BOX - side + 1))
        y = int(r.integers(0, CITY_BOX - side + 1))
        out.append((x, y, side, 15_000 >> (z - 10), k % 2 == 1))
    return out


BUCKETS = 256


def _ranges(q, off):
    """Index ranges of the bucketed points whose buckets meet the viewport."""
    x, y, side = q[0], q[1], q[2]
    cell = -(-CITY_BOX // BUCKETS)
    bx0, bx1 = x // cell, min(BUCKETS - 1, (x + side - 1) // cell)
    by0, by1 = y // cell, min(BUCKETS - 1, (y + side - 1) // cell)
    out = []
    for by in range(by0, by1 + 1):
        a, b = int(off[by * BUCKETS + bx0]), int(off[by * BUCKETS + bx1 + 1])
        if b > a:
            if out and out[-1][1] == a:
                out[-1] = (out[-1][0], b)
            else:
                out.append((a, b))
    return out or [(0, 0)]


def _points(case, seed):
    n = case["points"]
    if case.get("stars"):
        xy = _uniform_points(n, TINY_BOX, _gen(seed, 1))
        vals = torch.randint(100, 10_001, (n,), generator=_gen(seed, 2), device=DEV,
                             dtype=torch.int64)
    else:
        xy = _mixture_points(n, CITY_BOX, _gen(seed, 1))
        vals = _cents(n, _gen(seed, 2))
    return xy, (vals if case.get("values", True) else None)


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case, "old": []}
    if case.get("stars"):
        st["polys"] = _stars(case["stars"], TINY_BOX, _gen(seed, 3))
    else:
        st["polys"] = _city(case["polys"], _gen(seed, 3))
    if kind != "join":
        st["xy"], st["vals"] = _points(case, seed)
    eps = case.get("eps")
    if kind == "probe":
        st["h"] = sba.Approx(*st["polys"], eps)
    elif kind == "range":
        st["h"] = sba.Approx(*st["polys"], eps)
        i = st["h"].info()
        st["hb"] = sba.Approx(*st["polys"], eps, boundary_only=True, tile_log2=i["tile_log2"],
                              sub_log2=i["sub_log2"])
    elif kind in ("runs", "partitioned"):
        st["h"] = sba.Approx(*st["polys"], eps, kind="hilbert", search=case["search"],
                             log2_leaves=20)
        if kind == "partitioned":
            st["scratch"] = torch.empty(sba.Approx.scratch_bytes(case["points"], case["values"]),
                                        dtype=torch.uint8, device=DEV)
        elif case["ordered"]:
            st["xy"], st["vals"], _ = sba.bucket_points(st["xy"], st["vals"], 0, 0,
                                                        -(-CITY_BOX // 1024), 1024)
    elif kind == "viewports":
        st["xy"], st["vals"], off = sba.bucket_points(st["xy"], st["vals"], 0, 0,
                                                      -(-CITY_BOX // BUCKETS), BUCKETS)
        off = off.cpu().numpy()
        st["queries"] = [(q, _ranges(q, off)) for q in _viewports(case, seed)]
    elif kind == "pindex_build":
        ix = sba.PointIndex(st["xy"], st["vals"], eps)
        st["h"] = sba.Approx(*st["polys"], eps, kind="hilbert", key_grid=ix)
        ix.close()
    elif kind == "pindex_query":
        st["ix"] = sba.PointIndex(st["xy"], st["vals"], eps)
        del st["xy"], st["vals"]
    elif kind == "join":
        other = _city(case["polys2"], _gen(seed, 4))
        grid = sba.key_grid_for(eps, _Polys(st["polys"]), _Polys(other))
        st["h"] = sba.Approx(*st["polys"], eps, kind="hilbert", key_grid=grid)
        st["h2"] = sba.Approx(*other, eps, kind="hilbert", key_grid=grid)
        st["table"] = torch.empty((3, 16 * (case["polys"] + case["polys2"])), dtype=torch.int64,
                                  device=DEV)
    return st


def _retire(st, new):
    """Handles of the last pass: a build has synchronised the stream since
    their work was queued, so they go back without another wait."""
    for h in st["old"]:
        h.close(sync=False)
    st["old"] = new


def run(state):
    st, case = state, state["case"]
    kind = case["kind"]
    if kind == "step":
        h = sba.Approx(*st["polys"], case["eps"])
        _retire(st, [h])
        return h.aggregate(st["xy"], st["vals"])
    if kind == "probe":
        return st["h"].aggregate(st["xy"], st["vals"])
    if kind == "range":
        return sba.aggregate_range(st["h"], st["hb"], st["xy"], st["vals"])
    if kind == "runs":
        return st["h"].aggregate(st["xy"], st["vals"])
    if kind == "partitioned":
        return st["h"].aggregate_partitioned(st["xy"], st["vals"], scratch=st["scratch"])
    if kind == "viewports":
        handles, tasks, outs = [], [], []
        for (x, y, side, eps, with_sum), ranges in st["queries"]:
            h = sba.Approx(*st["polys"], eps, window=(x, y, x + side, y + side))
            handles.append(h)
            vals = st["vals"] if with_sum else None
            counts = torch.empty(h.n_polys, dtype=torch.int64, device=DEV)
            sums = torch.empty_like(counts) if with_sum else None
            outs.append((counts, sums))
            for a, b in ranges:
                tasks.append(sba.Task(h, st["xy"], vals, a, b, (x, y, side, side), counts, sums))
        sba.aggregate_batch(tasks)
        _retire(st, handles)
        return outs
    if kind == "pindex_build":
        ix = sba.PointIndex(st["xy"], st["vals"], case["eps"])
        _retire(st, [ix])
        return ix.aggregate(st["h"], "learned")
    if kind == "pindex_query":
        h = sba.Approx(*st["polys"], case["eps"], kind="hilbert", key_grid=st["ix"])
        _retire(st, [h])
        return st["ix"].aggregate(h, case["search"])
    # the pairs go to the program's own table, -1 past the last of them
    table = st["table"].fill_(-1)
    for row, col in zip(table, sba.join_pairs(st["h"], st["h2"])):
        row[:col.numel()] = col
    return table


def _vertices(polys):
    """Expected vertices of a partition's cells."""
    lo, hi = COARSE if polys < 1000 else FINE
    return polys * (4 + 2 * (lo + hi))


def work(case):
    """Input points (8 B) and values (8 B) once, polygon vertices (8 B) once,
    outputs once.  Kinds that answer from a standing structure alone count a
    key and a code (12 B) for each of its cells along the polygon edges."""
    kind = case["kind"]
    verts = 32 * case["stars"] if case.get("stars") else _vertices(case["polys"])
    polys = case["stars"] if case.get("stars") else case["polys"]
    per_point = 16 if case.get("values", True) else 8
    points = case.get("points", 0) * per_point
    out = polys * per_point
    s = max(1, int(case.get("eps", 2) / math.sqrt(2)))

    def edge_cells(k):  # both cells of a side keep the cells along it
        return 4.0 * math.sqrt(k) * CITY_BOX / s

    if kind in ("step", "pindex_build"):
        return {"bytes": 8 * verts + points + out}
    if kind in ("probe", "runs", "partitioned"):
        return {"bytes": points + out}
    if kind == "range":
        return {"bytes": points + 2 * out}
    if kind == "viewports":
        # a zoom level's square covers (40^(-(z-10)/8))^2 of the box
        share = sum(40.0 ** (-2 * _zoom(k) / 8.0) * 0.81 for k in range(case["queries"]))
        return {"bytes": case["queries"] * (8 * verts + 12 * polys)
                + share * case["points"] * 12}
    if kind == "pindex_query":
        return {"bytes": 8 * verts + 12 * edge_cells(polys) + out}
    return {"bytes": 12 * (edge_cells(polys) + edge_cells(case["polys2"])) + 16 * 2 * polys}


def exact(case, seed):
    """Counts, sums and cells are whole numbers: equal or wrong, with no
    rounding to measure."""
    return None
