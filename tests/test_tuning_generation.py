"""A tiling stored for other kernels is not applied (and not lost)."""
import json

import paper_2406_15236_amd as mpc
from paper_2406_15236_amd import tuning

TILING = {"tile_cells": 20, "grid": 3072, "yblock": 8, "order": 0}


class FakeSim:
    def __init__(self):
        self.params = [mpc.make_params(dict(L=(384, 384, 384), density=10.0))]
        self.calls = []

    def autotune(self, trial_steps):
        self.calls.append("autotune")

    def get_tiling(self):
        return dict(tile_cells=0, grid=141600, yblock=8, order=0, ntiles=566400)

    def set_tiling(self, *t):
        self.calls.append(("set_tiling", *t))


def test_entries_of_other_kernels_are_left_alone(tmp_path, monkeypatch):
    path = str(tmp_path / "cache.json")
    device = "gfx950/256cu"
    # as stored before the key named the kernels
    old = f"{device}|form0|flags0|384x384x384@10"
    json.dump({old: TILING}, open(path, "w"))
    sim = FakeSim()
    _, hit = tuning.autotune_cached(sim, 2, path=path, device=device)
    assert not hit and sim.calls == ["autotune"]
    assert json.load(open(path))[old] == TILING
    # and as a later generation will find today's
    monkeypatch.setattr(tuning, "KERNELS", "next")
    sim = FakeSim()
    assert not tuning.autotune_cached(sim, 2, path=path, device=device)[1]
    assert len(json.load(open(path))) == 3
    monkeypatch.undo()
    sim = FakeSim()
    assert tuning.autotune_cached(sim, 2, path=path, device=device)[1]
    assert sim.calls == [("set_tiling", 0, 141600, 8, 0)]
