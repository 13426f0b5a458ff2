"""Timed cases of the library: what its users have it do, at the sizes they do it.

The feature sets are those of ``paper_1403_0802_amd.synth`` (the stand-ins for the paper's
datasets), kept resident as a deployment keeps them:

* ``stars``   64 star polygons in the unit square (configuration 1);
* ``walks``   20,000 random-walk polylines in a 40 km plane, D = 50 m (configuration 2);
* ``regions`` the 5,000-polygon tessellation with holes, 1.5M vertices (configuration 3);
* ``roads``   200,000 random-walk polylines, 5.3M vertices, D = 100 m (configuration 4).

A case is one query (or one burst of served requests) of ``n`` points: ``op``, ``features``,
cell size, precision form and the grid's build-time options.  Points are drawn per seed on
the GPU, clustered as the configurations cluster them, with 1 in 500 outside the extent.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_1403_0802_amd import gp, synth

SIDE = {"stars": 1.0, "regions": 1.0, "walks": 40_000.0, "roads": 40_000.0}
RADIUS = {"walks": 50.0, "roads": 100.0}


def _case(name, op, features, n, cells, prec="mixed", prestage=0, lists=0):
    """``cells`` per side of the extent; ``lists`` = the option that keeps per cell only
    what can matter there (PIP: cell classes, P2P: segment lists)."""
    c = {"op": op, "features": features, "n": n, "cells": cells, "prec": prec,
         "prestage": prestage, "lists": lists}
    return {"name": name, **c} if name else c


def listed():
    return [
        # configuration 1 as it stands: a small FP64 point-in-polygon query, where the
        # chain of launches is the cost
        _case("pip_stars_fp64", "pip", "stars", 50_000, 64, "fp64"),
        # an interactive lookup of a screenful of positions in the region map
        _case("pip_lookup", "pip", "regions", 1_500, 512, prestage=1),
        # an ordinary request of the service (the middle of its 1K-4M range) on a grid with
        # every option on
        _case("pip_request", "pip", "regions", 250_007, 512, prestage=1, lists=1),
        # a first query on a grid built without options
        _case("pip_plain", "pip", "regions", 1_000_003, 512),
        # configuration 3 on the benchmark's grid: the large batch join
        _case("pip_batch", "pip", "regions", 50_000_000, 512, prestage=1),
        # a batch on a classified grid
        _case("pip_classes", "pip", "regions", 20_000_001, 512, prestage=1, lists=1),
        # configuration 2 as it stands: FP64 distances, few points per cell
        _case("p2p_walks_fp64", "p2p", "walks", 1_000_000, 400, "fp64"),
        # an interactive lookup of the nearest road
        _case("p2p_lookup", "p2p", "roads", 1_500, 200, prestage=1),
        # configuration 2's points in the mixed form on a grid without options
        _case("p2p_walks", "p2p", "walks", 999_983, 400),
        # map matching a day of positions with per-cell segment lists
        _case("p2p_lists", "p2p", "roads", 20_000_001, 400, lists=1),
        # configuration 4 on the benchmark's grid: the largest batch join
        _case("p2p_batch", "p2p", "roads", 200_000_000, 400, prestage=1),
        # configuration 5: a burst of requests of 1K-4M points, both operations, on the
        # continuous-batching server with captured graphs
        {"name": "serve_burst", "op": "serve", "n": 4_000_000, "requests": 16},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["pip"] * 5 + ["p2p"] * 5 + ["serve"])
    if op == "serve":
        return {"op": "serve", "n": _log_int(rng, 50_000, 4_000_000),
                "requests": rng.randint(4, 16)}
    prec = rng.choice(["mixed", "mixed", "mixed", "fp64"])
    options = rng.choice([(0, 0), (1, 0), (0, 1), (1, 1)])
    if op == "pip":
        features = rng.choice(["regions", "regions", "stars"])
        cells = rng.choice([256, 512] if features == "regions" else [32, 64, 100])
        top = 50_000_000 if features == "regions" else 2_000_000
        n = _log_int(rng, 1_000, min(top, 20_000_000) if prec == "fp64" else top)
    else:
        features = rng.choice(["roads", "roads", "walks"])
        cells = rng.choice([200, 400])
        top = 50_000_000 if features == "roads" else 4_000_000
        n = _log_int(rng, 1_000, min(top, 4_000_000) if prec == "fp64" else top)
    return _case(None, op, features, n, cells, prec, *options)


# ------------------------------------------------------------------- inputs


@functools.lru_cache(maxsize=None)
def _geometry(features):
    """The resident feature set: fixed, as a deployment's map is."""
    if features == "stars":
        return synth.config1(n_points=1).geom
    if features == "walks":
        return synth.config2(n_points=1).geom
    if features == "regions":
        return synth.config3_geometry()[0]
    return synth.config4_geometry()


def _points(features, n, seed):
    """Coordinates of ``n`` points on the GPU, clustered like the configuration's."""
    side = SIDE[features]
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    f64 = dict(dtype=torch.float64, device="cuda")
    if features == "stars":
        x, y = (torch.rand(n, generator=g, **f64) for _ in range(2))
    else:
        k = 32 if side > 1.0 else 1_000
        rng = np.random.default_rng([int(seed), 7])
        if side > 1.0:
            centres, sigma = rng.uniform(2_000.0, 38_000.0, (k, 2)), np.full(k, 500.0)
        else:
            centres = rng.uniform(0.0, 1.0, (k, 2))
            sigma = np.exp(rng.uniform(math.log(0.002), math.log(0.02), k))
        centres = torch.as_tensor(centres, **f64)
        sigma = torch.as_tensor(sigma, **f64)
        which = torch.randint(0, k, (n,), generator=g, device="cuda")
        s = sigma[which]
        x, y = (centres[which, c] + s * torch.randn(n, generator=g, **f64) for c in (0, 1))
        for v in (x, y):  # reflect at the sides of the extent
            v.abs_()
            torch.sub(side, (side - v).abs_(), out=v)
            v.clamp_(0.0, float(np.nextafter(side, 0.0)))
        if side == 1.0:  # 30% of the occurrences are scattered
            m = torch.rand(n, generator=g, device="cuda") < 0.3
            for v in (x, y):
                torch.where(m, torch.rand(n, generator=g, **f64), v, out=v)
    out = torch.rand(n, generator=g, device="cuda") < 0.002
    x[out] += side
    return x, y


def _grid(op, features, cells, prestage, lists):
    p = synth.GridParams(cell_size=SIDE[features] / cells, radius_D=RADIUS.get(features, 0.0),
                         x0=0.0, y0=0.0, nx=cells, ny=cells, prestage=prestage,
                         cell_classes=lists if op == "pip" else 0,
                         segment_filter=lists if op == "p2p" else 0)
    return gp.gp_build_grid(op, _geometry(features), p)


def _outputs(op, n):
    i = torch.empty(n, dtype=torch.int32, device="cuda")
    return (i, torch.empty(n, dtype=torch.float64, device="cuda") if op == "p2p" else None)


def _requests(case):
    """(operation, points) of the burst: sizes even in their logarithm from 1,000 up, the
    operations and the order of sizes mixed."""
    r = case["requests"]
    sizes = [int(1_000 * (case["n"] / 1_000) ** (k / (r - 1))) for k in range(r)]
    order = np.random.default_rng(r).permutation(r)
    return [("pip" if j % 2 else "p2p", sizes[k]) for j, k in enumerate(order)]


def prepare(case, seed):
    if case["op"] == "serve":
        pip = _grid("pip", "regions", 512, 1, 0)
        p2p = _grid("p2p", "roads", 200, 1, 0)
        srv = gp.Server(pip, p2p, n_slots=4, slot_points=1 << 22, mem_budget=8 << 30)
        reqs = [(op, *_points("regions" if op == "pip" else "roads", n, 100 * seed + k),
                 *_outputs(op, n)) for k, (op, n) in enumerate(_requests(case))]
        torch.cuda.synchronize()  # the server's streams read what this one wrote
        return {"case": case, "server": srv, "requests": reqs}
    op, n = case["op"], case["n"]
    grid = _grid(op, case["features"], case["cells"], case["prestage"], case["lists"])
    return {"case": case, "grid": grid, "xy": _points(case["features"], n, seed),
            "out": _outputs(op, n), "ws": gp.new_workspace(grid, n, case["prec"])}


def run(state):
    case = state["case"]
    if case["op"] == "serve":
        srv = state["server"]
        tickets = [srv.submit(*r) for r in state["requests"]]
        for t in tickets:
            srv.wait(t)
        return [[r[3], r[4]] for r in state["requests"]]
    x, y = state["xy"]
    out_id, out_dist = state["out"]
    if case["op"] == "pip":
        gp.gp_pip(state["grid"], x, y, out_id, case["prec"], state["ws"])
        return [out_id]
    gp.gp_p2p(state["grid"], x, y, out_id, out_dist, case["prec"], state["ws"])
    return [out_id, out_dist]


# ------------------------------------------------------------------- what it takes


def _work(op, features, n):
    """The points in, the results out and the features once; each point against the edges
    of one feature at least (6 operations a crossing test, 14 a distance)."""
    g = _geometry(features)
    bytes_ = n * (20 if op == "pip" else 28) + g.n_vertices * 16
    edges = g.n_vertices if op == "pip" else g.n_vertices - g.n_features
    return bytes_, n * (6 if op == "pip" else 14) * edges / g.n_features


def work(case):
    if case["op"] == "serve":
        parts = [(op, "regions" if op == "pip" else "roads", n) for op, n in _requests(case)]
    else:
        parts = [(case["op"], case["features"], case["n"])]
    b, f = zip(*(_work(*p) for p in parts))
    return {"bytes": float(sum(b)), "flops": float(sum(f))}


def _segments_by_cell(features, cells):
    """Start offsets and segments of the lists "segments whose box, expanded by the range,
    touches the cell", for a grid of ``cells`` per side, and the segments' endpoints."""
    geom, side, reach = _geometry(features), SIDE[features], RADIUS[features] * 1.001
    x, y = torch.as_tensor(geom.x, device="cuda"), torch.as_tensor(geom.y, device="cuda")
    first = torch.ones(len(geom.x), dtype=torch.bool)
    first[torch.as_tensor(geom.ring_vert_off[1:]) - 1] = False  # a line's last vertex
    a = first.nonzero().flatten().cuda()
    ends = torch.stack([x[a], y[a], x[a + 1], y[a + 1]], 1)
    cs = side / cells

    def span(u, v):
        lo = ((torch.minimum(u, v) - reach) / cs).floor().long()
        hi = ((torch.maximum(u, v) + reach) / cs).floor().long()
        return lo.clamp(0, cells - 1), hi.clamp(0, cells - 1)

    xl, xh = span(ends[:, 0], ends[:, 2])
    yl, yh = span(ends[:, 1], ends[:, 3])
    wide, count = xh - xl + 1, (xh - xl + 1) * (yh - yl + 1)
    seg = torch.repeat_interleave(torch.arange(len(a), device="cuda"), count)
    k = torch.arange(len(seg), device="cuda") - torch.repeat_interleave(
        count.cumsum(0) - count, count)
    cell = (yl[seg] + k // wide[seg]) * cells + xl[seg] + k % wide[seg]
    cell, order = cell.sort()
    start = torch.searchsorted(cell, torch.arange(cells * cells + 1, device="cuda"))
    return start, seg[order], ends


def exact(case, seed):
    """Distances in FP64 (projection onto the segment, clamped); ids are whole numbers and
    have no such value.  None beyond 4M points, where it takes too long."""
    if case["op"] != "p2p" or case["n"] > 4_000_000:
        return None
    px, py = _points(case["features"], case["n"], seed)
    cells, side = 400, SIDE[case["features"]]
    start, seg, ends = _segments_by_cell(case["features"], cells)
    best = torch.full_like(px, math.inf)
    inside = ((px >= 0) & (px < side) & (py >= 0) & (py < side)).nonzero().flatten()
    cs = side / cells
    c = (py[inside] / cs).long().clamp_(0, cells - 1) * cells + \
        (px[inside] / cs).long().clamp_(0, cells - 1)
    todo = start[c + 1] - start[c]
    upto = todo.cumsum(0)
    at, n = 0, len(inside)
    while at < n:  # as many points at a time as have 2^25 segments
        done = int(upto[at - 1]) if at else 0
        to = max(at + 1, int(torch.searchsorted(upto, done + (1 << 25))))
        w = torch.arange(at, min(to, n), device="cuda")
        own = torch.repeat_interleave(w, todo[w])
        k = torch.arange(len(own), device="cuda") - torch.repeat_interleave(
            upto[w] - todo[w] - done, todo[w])
        ax, ay, bx, by = ends[seg[start[c[own]] + k]].unbind(1)
        x, y = px[inside[own]], py[inside[own]]
        dx, dy = bx - ax, by - ay
        len2 = dx * dx + dy * dy
        t = ((x - ax) * dx + (y - ay) * dy) / torch.where(len2 > 0, len2, torch.ones_like(len2))
        t = t.clamp_(0.0, 1.0)
        d = torch.hypot(x - ax - t * dx, y - ay - t * dy)
        best.scatter_reduce_(0, inside[own], d, "amin")
        at = to
    best[best > RADIUS[case["features"]]] = math.inf
    return [None, best]
