"""Tiles of programs that are tuned, and of those that are not (needs an MI355X)."""
import json
import math

import numpy as np
import pytest

import synth
from tests.test_gpu_parity import hx  # noqa: F401  (fixture)
from tests.test_gpu_resident_switch import same, scene

pytestmark = pytest.mark.gpu


def small(option="plain", **kw):
    return [scene(70, 30, option, seed=k, **kw) for k in range(4)]


def cells_key(scs):
    return round(math.log2(sum(int(np.count_nonzero(sc.active == 1)) if sc.active is not None
                               else sc.n for sc in scs)))


@pytest.mark.parametrize("tile", [0, 1, 2, 3])
def test_a_cached_ensemble_tile_is_taken(hx, tmp_path, monkeypatch, tile):
    """The default of a small FP64 ensemble does not replace what the cache names, not even the
    default of other ensembles."""
    scs = small()
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({f"gfx950/ensemble/fp64/2^{cells_key(scs)}":
                                 {"tile": 200 + tile, "us": 1.0, "all_us": [1.0]}}))
    assert hx.Ensemble.from_scenarios(scs, "fp64").info()["tile"] == 0
    monkeypatch.setenv("HEXSV_TUNE_CACHE", str(cache))
    ens = hx.Ensemble.from_scenarios(scs, "fp64")
    assert (ens.info()["mode"], ens.info()["tile"]) == ("batched", tile)
    # the caller's choice goes before the cache's
    assert hx.Ensemble.from_scenarios(scs, "fp64", mode="batched").info()["tile"] == 0
    assert hx.Ensemble.from_scenarios(scs, "fp64", mode="batched", tile=2).info()["tile"] == 2
    assert hx.Ensemble.from_scenarios(scs, "fp64", mode="persistent").info()["tile"] == 0
