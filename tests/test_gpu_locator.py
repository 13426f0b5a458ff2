"""The locator (the grid's per-point index, which serves queries at the library default)
against the oracle and against the tiled refinement (which an explicit tuning selects), on
the same grids: ids and distances bit for bit, and the same counters.

The cases are those in which its build can go wrong: cells that are not divided, divided to
every depth and divided differently from their neighbours; points on the lines between
subcells and on the doubles next to them; chains of edges that leave and re-enter a
subcell's band; more near segments than the two a query keeps; and geometry for which a
grid has no locator.  Both sides evaluate the definition's FP64 expressions, so every
comparison is exact.
"""
import numpy as np
import pytest

import oracle
from paper_1403_0802_amd import synth
from tests import pins

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gp():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1403_0802_amd import gp as gpmod
    return gpmod


def line_points(rng, params, n, k=64):
    """Points on the lines of a k x k division of the cells, and next to them."""
    cs = params.cell_size
    x = params.x0 + cs / k * rng.integers(0, params.nx * k + 1, n)
    y = params.y0 + cs / k * rng.integers(0, params.ny * k + 1, n)
    free = rng.integers(0, 3, n)
    x = np.where(free == 1, params.x0 + cs * params.nx * rng.uniform(0, 1, n), x)
    y = np.where(free == 2, params.y0 + cs * params.ny * rng.uniform(0, 1, n), y)
    step = rng.integers(-1, 2, (2, n))
    for v, s in ((x, step[0]), (y, step[1])):
        v[:] = np.where(s > 0, np.nextafter(v, np.inf), np.where(s < 0, np.nextafter(v, -np.inf), v))
    return x, y


def check(gp, kind, geom, params, px, py):
    og = oracle.build_grid(geom, params)
    if kind == "pip":
        want = (oracle.pip(geom, px, py, og),)
    else:
        want = oracle.p2p(geom, px, py, params.radius_D, og)
    x, y = torch.from_numpy(np.ascontiguousarray(px)).cuda(), torch.from_numpy(
        np.ascontiguousarray(py)).cuda()
    lists = "cell_classes" if kind == "pip" else "segment_filter"
    for options in ({}, {"prestage": 1}, {lists: 1}):
        grid = gp.gp_build_grid(kind, geom, synth.GridParams(**{**params.__dict__, **options}))
        for prec in ("fp64", "mixed"):
            gp.gp_reset_tuning(grid, prec)
            got = gp.run(grid, x, y, prec, stats=True)
            gp.gp_set_tuning(grid, prec, **gp.gp_get_tuning(grid, prec))
            tiled = gp.run(grid, x, y, prec, stats=True)
            for a, b, w in zip(got[:-1], tiled[:-1], want):
                bad = np.flatnonzero(a.cpu().numpy() != w)
                assert bad.size == 0, (kind, options, prec, bad.size, px[bad[:3]], py[bad[:3]])
                assert torch.equal(a, b), (kind, options, prec)
            for key in ("n_points", "n_paired", "tests", "tests_avoided"):
                assert got[-1][key] == tiled[-1][key], (kind, options, prec, key)


def comb(rng, teeth):
    """A polygon whose right side is a comb: chains that enter and leave every band."""
    y = np.sort(rng.uniform(0.05, 0.95, 2 * teeth))
    x = np.where(np.arange(2 * teeth) % 2 == 0, 0.9, rng.uniform(0.3, 0.8, 2 * teeth))
    return [(0.1, 0.05)] + [(0.95, 0.05)] + list(zip(x, y)) + [(0.95, 0.96), (0.1, 0.96)]


@pytest.mark.parametrize("cells", [1, 3, 16, 100])
def test_pip(gp, cells):
    """Stars, a comb, holes, horizontal and duplicate edges, from one cell that holds
    everything (divided 64 x 64) to cells of a few edges."""
    rng = np.random.default_rng(100 + cells)
    t = np.sort(rng.uniform(0, 2 * np.pi, 3000))
    sq = pins.box(0.2, 0.2, 0.8, 0.8)
    g = pins.polygons([
        [comb(rng, 60)],
        [sq, pins.box(0.3, 0.3, 0.7, 0.7, ccw=False)],
        [list(zip(0.5 + 0.4 * np.cos(t), 0.5 + 0.4 * np.sin(t)))],
        [sq + sq],  # every edge twice: even everywhere
        [pins.box(0.0, 0.5, 1.0, 0.75)],
        [pins.box(-1.0, -1.0, 2.0, 2.0)]])
    params = synth.GridParams(cell_size=1.0 / cells, x0=0.0, y0=0.0, nx=cells, ny=cells)
    px, py = rng.uniform(-0.05, 1.05, (2, 20_000))
    lx, ly = line_points(rng, params, 20_000)
    k = rng.integers(0, len(g.x), 4_000)  # on vertices, and level with vertices
    px = np.concatenate([px, lx, g.x[k[:2000]], rng.uniform(0, 1, 2000)])
    py = np.concatenate([py, ly, g.y[k[:2000]], g.y[k[2000:]]])
    check(gp, "pip", g, params, px, py)


@pytest.mark.parametrize("cells,off", [(1, 0.0), (7, 1e4), (40, -1e6), (40, 1e11)])
def test_p2p(gp, cells, off):
    """Random walks with repeated polylines, a star of 300 rays from one vertex and long
    segments, at several cell sizes and offsets; at an offset of 1e11 cells of 0.25 are
    below the locator's precision and the grid goes without one."""
    rng = np.random.default_rng(200 + cells)
    lines = []
    for _ in range(60):
        p = rng.uniform(0, 10, 2) + np.cumsum(rng.normal(0, 0.4, (int(rng.integers(2, 30)), 2)), 0)
        lines += [p] * int(rng.integers(1, 4))
    a = rng.uniform(0, 2 * np.pi, 300)
    lines += [np.array([(5.0, 5.0), (5.0 + 2 * np.cos(t), 5.0 + 2 * np.sin(t))]) for t in a]
    lines += [np.array([(-50.0, -49.0), (60.0, 61.5)]), np.array([(2.0, 2.0)] * 3)]
    g = pins.polylines([[(x + off, y + off) for x, y in p] for p in lines])
    cs = 10.0 / cells
    for D in (0.0, 0.3, 20.0):
        params = synth.GridParams(cell_size=cs, radius_D=D, x0=off, y0=off, nx=cells, ny=cells)
        px, py = off + rng.uniform(-0.5, 10.5, (2, 5_000))
        lx, ly = line_points(rng, params, 5_000, 32)
        k = rng.integers(0, len(g.x), 1_000)
        px = np.concatenate([px, lx, g.x[k], np.full(5, off + 5.0)])
        py = np.concatenate([py, ly, g.y[k], np.full(5, off + 5.0)])
        check(gp, "p2p", g, params, px, py)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 4099])
def test_sizes_and_capture(gp, n):
    """Every remainder of a wave and a workgroup, captured in a graph and replayed on new
    points with eager calls between."""
    rng = np.random.default_rng(n)
    wp = synth.config1(n_points=4 * n, grid_n=3, seed_salt=n)
    wl = synth.config2(n_points=4 * n, n_lines=300, seed_salt=n)
    for w in (wp, wl):
        grid = gp.gp_build_grid(w.kind, w.geom, w.params)
        pts = [torch.from_numpy(np.ascontiguousarray(v)).cuda().view(4, n) for v in (w.px, w.py)]
        x, y = pts[0][0].clone(), pts[1][0].clone()
        out = torch.empty(n, dtype=torch.int32, device="cuda")
        dist = torch.empty(n, dtype=torch.float64, device="cuda")
        ws = gp.new_workspace(grid, n, "mixed")

        def query():
            if w.kind == "pip":
                gp.gp_pip(grid, x, y, out, "mixed", ws)
            else:
                gp.gp_p2p(grid, x, y, out, dist, "mixed", ws)
        query()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            query()
        for r in range(4):
            x.copy_(pts[0][r]), y.copy_(pts[1][r])
            out.fill_(-9), dist.fill_(-9.0)
            graph.replay()
            got = out.clone(), dist.clone()
            query()
            torch.cuda.synchronize()
            assert torch.equal(got[0], out) and torch.equal(got[1], dist)
            og = oracle.build_grid(w.geom, w.params)
            px, py = (p[r].cpu().numpy() for p in pts)
            if w.kind == "pip":
                assert np.array_equal(out.cpu().numpy(), oracle.pip(w.geom, px, py, og))
            else:
                wid, wd = oracle.p2p(w.geom, px, py, w.params.radius_D, og)
                assert np.array_equal(out.cpu().numpy(), wid)
                assert np.array_equal(dist.cpu().numpy(), wd)


def test_default_stream_is_the_current_one(gp):
    """A call without a stream runs on torch's current one, also inside a stream context."""
    s = torch.cuda.Stream()
    assert gp._current_stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(s):
        assert gp._current_stream() == s.cuda_stream
    assert gp._current_stream() == torch.cuda.current_stream().cuda_stream


@pytest.mark.parametrize("graphs", [True, False])
def test_served_while_the_tuning_changes(gp, graphs):
    """One server, its blocks and their captured graphs reused while the grids go from the
    locator to the tiled refinement and back: every request equals the oracle, and counts
    the same tests on either path."""
    wp = synth.config1(n_points=9_000, grid_n=3, seed_salt=5)
    wl = synth.config2(n_points=9_000, n_lines=300, seed_salt=5)
    grids = [gp.gp_build_grid(w.kind, w.geom, w.params) for w in (wp, wl)]
    og = [oracle.build_grid(w.geom, w.params) for w in (wp, wl)]
    srv = gp.Server(*grids, n_slots=2, slot_points=4096, mem_budget=1 << 30, use_graphs=graphs)
    tests = []
    for step, n in enumerate((9_000, 3_000, 1, 9_000, 2_000)):
        for g in grids:
            gp.gp_reset_tuning(g, "mixed")
            if step in (1, 3):
                gp.gp_set_tuning(g, "mixed", **gp.gp_get_tuning(g, "mixed"))
        before = srv.stats()["tests"]
        for w, o in zip((wp, wl), og):
            px, py = w.px[-n:], w.py[-n:]
            x, y = (torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in (px, py))
            out = torch.full((n + 8,), -9, dtype=torch.int32, device="cuda")
            dist = torch.full((n + 8,), -9.0, dtype=torch.float64, device="cuda")
            torch.cuda.synchronize()
            if w.kind == "pip":
                srv.wait(srv.submit("pip", x, y, out))
                want = oracle.pip(w.geom, px, py, o), None
            else:
                srv.wait(srv.submit("p2p", x, y, out, dist))
                want = oracle.p2p(w.geom, px, py, w.params.radius_D, o)
                assert np.array_equal(dist[:n].cpu().numpy(), want[1]), (step, n)
            assert np.array_equal(out[:n].cpu().numpy(), want[0]), (w.kind, step, n)
            assert bool((out[n:] == -9).all()) and bool((dist[n:] == -9.0).all())
        tests.append(srv.stats()["tests"] - before)
    assert tests[0] == tests[3] > 0
    srv.close()
