"""The tiled refinement under the tests that describe it.

At the library default a grid's queries run on its locator, and so do most tests of the parity,
random and serving files.  Here the same tests run with every grid set to the tiled
refinement's default configuration, and each query is checked to have taken that path; the
rules for untuned grids run on grids that have no locator.
"""
import numpy as np
import pytest

import oracle
from paper_1403_0802_amd import synth
from tests import golden_cases
from tests import test_gpu_parity as parity
from tests import test_gpu_random as rnd
from tests import test_gpu_serving as serving
from tests import test_zz_no_alloc as no_alloc
from tests.test_gpu_serving import setup  # noqa: F401  (a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


class Tiled:
    """The binding with grids that start out, and are reset, to an explicit tuning: the tiled
    refinement's default.  ``rechecked`` counts the points recomputed in FP64."""

    def __init__(self, gp):
        self._gp = gp
        self.queries = self.rechecked = 0

    def __getattr__(self, name):
        return getattr(self._gp, name)

    def gp_build_grid(self, *a, **k):
        grid = self._gp.gp_build_grid(*a, **k)
        for prec in ("fp64", "mixed"):
            self.gp_reset_tuning(grid, prec)
        return grid

    def gp_reset_tuning(self, grid, prec):
        self._gp.gp_reset_tuning(grid, prec)
        self._gp.gp_set_tuning(grid, prec, **self._gp.gp_get_tuning(grid, prec))

    def run(self, *a, stats=False, **k):
        out = self._gp.run(*a, stats=True, **k)
        st = out[-1]
        # the locator sorts no points
        assert st["ms_pairing"] > 0.0 or st["n_points"] == 0, st
        self.queries += st["n_points"] > 0
        self.rechecked += st["n_rechecked"]
        if stats:
            return out
        return out[0] if len(out) == 2 else out[:-1]


@pytest.fixture(scope="module")
def gp():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_1403_0802_amd import gp as gpmod
    return gpmod


@pytest.fixture
def tiled(gp):
    t = Tiled(gp)
    yield t
    assert t.queries > 0


@pytest.fixture(scope="module")
def c1():
    w = synth.config1()
    return w, oracle.run(w)[1]


@pytest.fixture(scope="module")
def c2():
    w = synth.config2()
    return (w, *oracle.run(w)[1:])


@pytest.fixture(scope="module")
def c3_geom():
    return synth.config3_geometry()


@pytest.mark.parametrize("case", ["c1", "c2", "c2_derived", "on_lines", "exact_lines"])
def test_pairing(tiled, case):
    parity.test_pairing_bit_exact(tiled, case)


@pytest.mark.parametrize("prec,pre", [("fp64", 0), ("mixed", 0), ("mixed", 1)])
def test_pip_c1(tiled, c1, prec, pre):
    parity.test_pip_c1(tiled, c1, prec, pre)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_p2p_c2(tiled, c2, prec):
    parity.test_p2p_c2(tiled, c2, prec)


@pytest.mark.parametrize("name", golden_cases.ALL)
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_golden(tiled, name, prec):
    parity.test_golden_fixtures(tiled, name, prec)


def test_shuffle(tiled):
    parity.test_shuffle_invariance(tiled)


def test_empty_and_unpaired(tiled):
    parity.test_empty_and_unpaired_inputs(tiled)


def test_holes_overlaps_and_long_rings(tiled):
    parity.test_holes_overlaps_and_long_rings(tiled)


def test_cell_classes_counts_and_ids(tiled):
    parity.test_pip_cell_classes_counts_and_ids(tiled)


@pytest.mark.parametrize("case", ["c1", "holes", "c3"])
def test_cell_classes(tiled, c1, c3_geom, case):
    parity.test_pip_cell_classes_equal_unclassified(tiled, c1, c3_geom, case)


@pytest.mark.parametrize("kind", ["pip", "p2p"])
def test_cell_size(tiled, c1, kind):
    parity.test_results_invariant_under_cell_size(tiled, c1, kind)


@pytest.mark.parametrize("case", ["c2", "ties", "near", "c4"])
def test_segment_filter(tiled, case):
    parity.test_p2p_segment_filter_equal_unfiltered(tiled, case)


@pytest.mark.parametrize("case", ["c2", "ties", "near", "c4"])
def test_prestage(tiled, case):
    parity.test_p2p_prestage_equal_plain(tiled, case)
    assert case != "c4" or tiled.rechecked > 0  # three polylines near a tie


def test_near_edges(tiled):
    parity.test_near_edge_sweep_mixed(tiled)
    assert tiled.rechecked > 0


def test_ties_range_and_degenerate_segments(tiled):
    parity.test_p2p_ties_range_and_degenerate_segments(tiled)


def test_equidistant_segments(tiled):
    parity.test_p2p_exact_pass_many_equidistant_segments(tiled)


def test_near_range_and_near_ties(tiled):
    parity.test_p2p_near_range_and_near_tie_sweep(tiled)


def test_derived_extent_and_single_cell(tiled):
    parity.test_derived_extent_and_single_cell(tiled)


def test_c3_mixed_equals_fp64(tiled, c3_geom):
    parity.test_c3_mixed_equals_fp64_and_oracle_sample(tiled, c3_geom)


def test_c4_mixed_equals_fp64(tiled):
    parity.test_c4_scaled_mixed_vs_oracle_sample(tiled)


def test_c3_full_size(tiled, c3_geom):
    """50M points on the kernel that the benchmark times."""
    parity.test_c3_full_size_50m(tiled, c3_geom, "bench")


def test_c4_full_size(tiled):
    """200M points on the kernel that the benchmark times."""
    parity.test_c4_full_size_200m(tiled, "bench")


@pytest.mark.parametrize("seed", rnd.SEEDS)
def test_random_pip(tiled, seed):
    rnd.test_random_pip_equals_oracle(tiled, seed)


@pytest.mark.parametrize("seed", rnd.SEEDS)
def test_random_p2p(tiled, seed):
    rnd.test_random_p2p_equals_oracle(tiled, seed)


def test_signed_zeros(tiled):
    rnd.test_signed_zero_coordinates(tiled)


@pytest.mark.parametrize("seed", range(3))
def test_pip_item_sizes(tiled, seed):
    rnd.test_pip_item_sizes(tiled, seed)


@pytest.mark.parametrize("seed", range(2))
def test_p2p_item_sizes(tiled, seed):
    rnd.test_p2p_item_sizes(tiled, seed)


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("kind", ["pip", "p2p"])
def test_noalloc(tiled, kind, prec):
    no_alloc.test_noalloc_equals_workspace_entry_points(tiled, kind, prec)


# ---------------------------------------------------------------- serving


@pytest.fixture
def served(setup):  # noqa: F811
    gp, g3, g4, reqs, want = setup
    t = Tiled(gp)
    for g in (g3, g4):
        t.gp_reset_tuning(g, "mixed")
        # device inputs alone, through the direct entry point: the path that is served
        k = next(r for r in reqs if gp.KINDS[r[0]] == g.kind)
        t.run(g, k[1], k[2], "mixed")
    yield t, g3, g4, reqs, want
    for g in (g3, g4):
        gp.gp_reset_tuning(g, "mixed")


@pytest.mark.parametrize("graphs", [True, False])
def test_served_mix(served, graphs):
    serving.test_mix_equals_alone(served, graphs)


def test_served_prestaged_grid(served):
    serving.test_prestaged_grid_in_the_mix(served)


def test_served_host_inputs(served):
    serving.test_host_inputs_and_tight_budget(served)


def test_served_admission(served):
    serving.test_admission_waits_for_memory_not_streams(served)


def test_served_large_request(served):
    serving.test_large_request_spreads_over_free_streams(served)


# ---------------------------------------------------------------- untuned, no locator


def with_outlier(w):
    """The workload with one more feature so far out that its grid goes without a locator,
    and that no point can meet."""
    g = w.geom
    at = 1e155 if w.kind == "pip" else 2.0 ** 32 * w.params.cell_size
    ox, oy = at * np.array([1.0, 1.25, 1.0]), at * np.array([1.0, 1.0, 1.25])
    off = np.append(g.ring_vert_off, g.ring_vert_off[-1] + 3)
    rings = None if g.feature_ring_off is None else np.append(g.feature_ring_off,
                                                              g.feature_ring_off[-1] + 1)
    return synth.Geometry(g.kind, off, np.append(g.x, ox), np.append(g.y, oy), rings)


@pytest.mark.parametrize("kind", ["pip", "p2p"])
def test_untuned_grid_without_a_locator(gp, kind):
    """The default's own rules: few points (one workgroup per item), few points per cell (at
    most two per lane) and enough of both for the persistent queue and four per lane."""
    n = (1 << 22) + 77
    w = (synth.config1(n_points=n, grid_n=3, seed_salt=9) if kind == "pip"
         else synth.config2(n_points=n, n_lines=2_000, seed_salt=9))
    geom = with_outlier(w)
    og = oracle.build_grid(geom, w.params)
    want = (oracle.pip(geom, w.px, w.py, og),) if kind == "pip" else oracle.p2p(
        geom, w.px, w.py, w.params.radius_D, og)
    x, y = torch.from_numpy(w.px).cuda(), torch.from_numpy(w.py).cuda()
    lists = "cell_classes" if kind == "pip" else "segment_filter"
    for options in ({}, {"prestage": 1}, {lists: 1}):
        grid = gp.gp_build_grid(kind, geom, synth.GridParams(**{**w.params.__dict__, **options}))
        for prec in ("fp64", "mixed"):
            for m in (1, 63, 4_099, 300_001, n):
                got = gp.run(grid, x[:m], y[:m], prec, stats=True)
                assert got[-1]["ms_pairing"] > 0.0, "the grid has a locator"
                for a, b in zip(got, want):
                    assert np.array_equal(a.cpu().numpy(), b[:m]), (options, prec, m)
