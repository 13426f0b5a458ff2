"""bench.py --cell-sweep without a GPU: each size is timed on the headline's path (an explicit
tuning) as well as on the library's default path, and the best size is the headline's."""
import json

import numpy as np
import torch

import bench
from paper_1403_0802_amd import synth


class Grid:
    def __init__(self, params):
        self.p, self.tuned = params, None

    def info(self):
        return {"nx": self.p.nx, "ny": self.p.ny, "n_pairs": 7, "device_bytes": 100}


class Binding:
    """Queries of tuned grids take 1 ms at cells of 50 m and 1/256 and 2 ms elsewhere; untuned
    ones 0.1 ms, least (0.05) at 400 m and 1/2048."""

    def gp_build_grid(self, kind, geom, params):
        return Grid(params)

    def new_workspace(self, grid, n, prec, device):
        return None

    def gp_get_tuning(self, grid, prec):
        return {"points_per_lane": 4, "persistent": 1}

    def gp_set_tuning(self, grid, prec, **t):
        grid.tuned = t

    def run(self, grid, x, y, prec, ws=None, stats=False):
        cs = grid.p.cell_size
        if grid.tuned is None:
            ms = 0.05 if cs in (400.0, 1 / 2048) else 0.1
        else:
            ms = 1.0 if cs in (50.0, 1 / 256) else 2.0
        return None, {"ms_total": ms, "tests": 5}


def test_the_sweep_times_the_headline_path(capsys, monkeypatch):
    monkeypatch.setattr(torch.cuda, "empty_cache", lambda: None)
    v = np.zeros(300)
    c3 = (None, synth.GridParams(**bench.PIP_GRID), v, v)
    c4 = (None, synth.GridParams(**bench.P2P_GRID), v, v)
    bench.cell_sweep(Binding(), torch, "cpu", c3, c4)
    out = json.loads(capsys.readouterr().out)["cell_sweep"]
    for name, best, sizes in (("pip_c3", 1 / 256, 5), ("p2p_c4", 50.0, 5)):
        rows = out[name]["rows"]
        assert out[name]["best_cell_size"] == best and len(rows) == sizes
        assert all(r["ms"] >= 1.0 and r["ms_locator"] <= 0.1 for r in rows)
