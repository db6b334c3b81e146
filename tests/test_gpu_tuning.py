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


@pytest.mark.parametrize("nq,nr,precision,option", [
    (64, 64, "fp64", "plain"), (512, 512, "fp32", "plain"), (512, 512, "fp64", "masked"),
    (300, 300, "fp32", "viscous"), (1000, 1000, "fp32", "plain")])
def test_a_tuned_simulation_still_runs_on_chip(hx, tmp_path, nq, nr, precision, option):
    """The tuner times what run() would do: the on-chip launches are the fastest here by a
    third and more, so whichever variant wins is one of theirs."""
    print(f"[tuned {nq}x{nr} {precision} {option}]", flush=True)
    sc = scene(nq, nr, option)
    sim = hx.Sim.from_scenario(sc, precision)
    sim.run(1e9, max_steps=30)
    before = sim.state_numpy(), sim.books()
    n = sim.resident_launches()
    cache = str(tmp_path / "tune.json")
    tile, ms = sim.autotune(nlaunch=30, cache_path=cache)
    same((sim.state_numpy(), sim.books()), before, "left unchanged")
    assert sim.resident_launches() == n and sim.info()["tile"] == tile
    sim.run(1e9, max_steps=100)
    assert sim.resident_launches() > n
    times = next(iter(json.load(open(cache)).values()))["all_us"]
    assert times[tile] == min(times) and abs(times[tile] - 1e3 * ms) <= 1e-3 * times[tile]
    if precision == "fp64":  # every tile and path the same state
        ref = hx.Sim.from_scenario(sc, precision)
        ref.set_resident(False)
        ref.run(1e9, max_steps=30)
        ref.run(1e9, max_steps=100)
        a, b = sim.state_numpy(), ref.state_numpy()
        assert all(np.array_equal(a[k], b[k]) for k in a)


@pytest.mark.parametrize("precision,option", [("fp64", "plain"), ("fp64", "viscous"),
                                              ("fp32", "plain"), ("fp32", "viscous")])
def test_a_tuned_ensemble_still_runs_on_chip(hx, precision, option):
    scs = small(option)
    ens = hx.Ensemble.from_scenarios(scs, precision)
    ens.run(1e9, max_steps=30)
    before = [(ens.state_numpy(k), ens.books(k)) for k in range(len(scs))]
    n = ens.resident_launches()
    assert n > 0
    code, _ = ens.autotune(ksteps=5)
    assert code // 100 == 2 and ens.resident_launches() == n
    for k in range(len(scs)):
        same((ens.state_numpy(k), ens.books(k)), before[k], k)
    ens.run(1e9, max_steps=100)
    assert ens.resident_launches() > n


def test_tuning_with_the_switch_off_times_single_launches(hx):
    """What run() would do is a launch per step then, for any variant."""
    sim = hx.Sim.from_scenario(scene(64, 64, "plain"), "fp64")
    sim.run(1e9, max_steps=30)
    _, on_chip = sim.autotune(nlaunch=30)
    sim.set_resident(False)
    _, single = sim.autotune(nlaunch=30)
    assert on_chip < single
