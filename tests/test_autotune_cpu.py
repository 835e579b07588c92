"""The tuner's cache of tile heights: an entry is installed only if it was
measured on the kernels that the heights would be used for."""
import json
from types import SimpleNamespace

import torch

from paper_2502_05279_amd import autotune, boxmg


def test_heights_of_other_kernels_are_measured_again(tmp_path, monkeypatch):
    path = tmp_path / "tile_rows.json"
    path.write_text(json.dumps({"gfx950:fp64:7": {"rows": 64, "ms": {"64": 1.0}}}))
    monkeypatch.setenv("BMG_TUNE_CACHE", str(path))
    monkeypatch.setattr(autotune, "_arch", lambda: "gfx950")
    monkeypatch.setattr(boxmg, "discretize", lambda k, f: (k, f))
    monkeypatch.setattr(autotune, "torch", SimpleNamespace(device=lambda name: "cpu", from_numpy=torch.from_numpy))
    timed, installed = [], {}
    monkeypatch.setattr(autotune, "_time_level", lambda st, rhs, level, rows, *a: timed.append(rows) or 1.0 / rows)
    monkeypatch.setattr(boxmg, "tile_rows_set", installed.__setitem__)
    for again in (False, True):          # the entry it writes is its own and is taken
        timed.clear()
        assert autotune.tune(sizes=(7,), candidates=(2, 4)) == {7: 4} == installed
        assert bool(timed) != again
