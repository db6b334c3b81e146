"""On-chip launches that are given up: nothing of them is kept, single launches take over after
the last committed step, and the failing cell is the one that single launches name (needs an
MI355X)."""
import threading

import numpy as np
import pytest
import torch

import synth
from tests.test_gpu_parity import hx  # noqa: F401  (fixture)
from tests.test_gpu_resident_switch import same, scene

pytestmark = pytest.mark.gpu


def run(sim, *steps):
    for n in steps:
        sim.run(1e9, max_steps=n)
    return sim.state_numpy(), sim.books()


@pytest.mark.parametrize("launch", [0, 1, 3])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nq,nr,tile,option", [(200, 190, 0, "masked"), (130, 1100, 0, "masked"),
                                                (1000, 1000, 2, "plain")])
def test_single_launches_take_over(hx, nq, nr, tile, option, precision, launch):
    """Launch 0, 1 or 3 of the five queued for 450 steps misses a workgroup: the others' waits
    run out, nothing of it is kept, and single steps do what is left after the five."""
    print(f"[given up {nq}x{nr} tile {tile} {precision} launch {launch}]", flush=True)
    sc = scene(nq, nr, option)
    ref = hx.Sim.from_scenario(sc, precision, tile=tile)
    ref.set_resident(False)
    want = run(ref, 7, 450)
    sim = hx.Sim.from_scenario(sc, precision, tile=tile)
    sim.run(1e9, max_steps=7)
    n0 = sim.resident_launches()
    hx._check(hx.lib().hexsv_sim_drop_resident(sim._h, launch))
    same(run(sim, 450), want, launch)
    assert sim.resident_launches() == n0 + 5
    # the next run goes without, the one after it on chip again
    same(run(sim, 60), run(ref, 60), "remembered")
    assert sim.resident_launches() == n0 + 5
    same(run(sim, 130), run(ref, 130), "on chip again")
    assert sim.resident_launches() == n0 + 7


def test_runs_without_grow_while_it_goes_on(hx):
    sim = hx.Sim.from_scenario(scene(64, 16, "plain"), "fp32")
    tried = []
    for _ in range(15):
        hx._check(hx.lib().hexsv_sim_drop_resident(sim._h, 0))
        n = sim.resident_launches()
        sim.run(1e9, max_steps=1)
        tried.append(sim.resident_launches() > n)
    assert [k for k, t in enumerate(tried) if t] == [0, 2, 6, 14]


@pytest.mark.parametrize("scenario,launch", [(0, 0), (3, 0), (3, 2), (5, 1)])
@pytest.mark.parametrize("precision,tile", [("fp32", 2), ("fp64", 0), ("fp32", 0)])
def test_one_scenario_gives_up(hx, precision, tile, scenario, launch):
    sizes = [(1, 1), (64, 16), (65, 17), (130, 40), (30, 100), (200, 13)]
    scs = [scene(nq, nr, "masked", seed=k) for k, (nq, nr) in enumerate(sizes)]
    ends = [1.0 + 0.3 * k for k in range(len(scs))]
    print(f"[given up by scenario {scenario}, launch {launch} {precision} tile {tile}]", flush=True)
    out = []
    for on in (False, True):
        ens = hx.Ensemble.from_scenarios(scs, precision, mode="batched", tile=tile)
        ens.set_resident(on)
        ens.run(ends)
        n0 = ens.resident_launches()
        if on:
            hx._check(hx.lib().hexsv_ensemble_drop_resident(ens._h, scenario, launch))
        ens.run(1e9, max_steps=310)
        n1 = ens.resident_launches()
        ens.run(1e9, max_steps=20)  # remembered
        n2 = ens.resident_launches()
        ens.run(1e9, max_steps=20)
        n3 = ens.resident_launches()
        assert (n1 - n0, n2 - n1, n3 - n2) == ((4, 0, 1) if on else (0, 0, 0))
        out.append([(ens.state_numpy(k), ens.books(k)) for k in range(len(scs))])
    for k in range(len(scs)):
        same(out[0][k], out[1][k], k)


def flood(precision, nq=150, nr=70):
    """Still water for about 145 steps before t = 0; then rain under which the water column of
    one cell, the one of porosity 0.1, leaves the number range in one step."""
    n, bad = nq * nr, 31 * nq + 77
    th = np.ones(n)
    th[bad] = 0.1
    sc = synth.c1_planar(nq, nr, t_end=1e9)
    return bad, sc.with_(z=np.zeros(n), theta=th, alpha_p=np.zeros(n), h0=np.full(n, 0.01),
                         side=(synth.WALL,) * 4, rain_kind=0, i_a=3e38 if precision == "fp32" else 1.7e308)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_the_failing_cell_is_named(hx, precision):
    bad, sc = flood(precision)
    out = []
    for on in (True, False):
        sim = hx.Sim.from_scenario(sc, precision)
        sim.set_state(sc.h0, sc.v10, sc.v20, -100.0)
        sim.set_resident(on)
        with pytest.raises(hx.HexsvError) as e:
            sim.run(1e9)
        assert e.value.code == hx.ENUMERIC and f"cell {bad} " in str(e.value)
        assert (sim.resident_launches() > 0) == on
        out.append((sim.state_numpy(), sim.books(), str(e.value)))
    assert out[0][1]["steps"] > 100 and out[0][2] == out[1][2]
    same(out[0], out[1], precision)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_the_failing_scenario_is_named(hx, precision):
    bad, sc = flood(precision)
    scs = [scene(65, 17, "masked", seed=k) for k in range(3)]
    out = []
    for on in (True, False):
        ens = hx.Ensemble.from_scenarios(scs[:1] + [sc] + scs[1:], precision, mode="batched", tile=0)
        ens.set_scenario(1, sc, -100.0)
        ens.set_resident(on)
        with pytest.raises(hx.HexsvError) as e:
            ens.run(1e9, max_steps=400)
        assert e.value.code == hx.ENUMERIC and "scenario 1 at cell" in str(e.value)
        assert (ens.resident_launches() > 0) == on
        out.append((ens.state_numpy(1), ens.books(1)))
    assert out[0][1]["steps"] > 100
    same(out[0], out[1], precision)


@pytest.mark.parametrize("nq,nr", [(200, 190), (512, 512)])
def test_two_streams_at_once(hx, nq, nr):
    """Two threads, each with a simulation and an ensemble on a stream of its own, compete for
    the compute units: whatever is given up, the results are those of a run alone."""
    scs = [scene(nq, nr, "masked", seed=s) for s in (1, 2)]
    small = [scene(130, 40, "plain", seed=s) for s in range(4)]
    want = []
    for sc in scs:
        sim = hx.Sim.from_scenario(sc, "fp32")
        sim.set_resident(False)
        want.append(run(sim, *[100] * 4))
    ref = hx.Ensemble.from_scenarios(small, "fp64")
    ref.set_resident(False)
    ref.run(1e9, max_steps=400)
    want_ens = [(ref.state_numpy(k), ref.books(k)) for k in range(4)]
    got, ens_got, err = [None, None], [None, None], []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                sim = hx.Sim.from_scenario(scs[i], "fp32")
                ens = hx.Ensemble.from_scenarios(small, "fp64")
                for _ in range(4):
                    sim.run(1e9, max_steps=100)
                    ens.run(1e9, max_steps=100)
                got[i] = sim.state_numpy(), sim.books()
                ens_got[i] = [(ens.state_numpy(k), ens.books(k)) for k in range(4)]
        except Exception as e:  # noqa: BLE001  (reported by the main thread)
            err.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not err, err
    for i in (0, 1):
        same(got[i], want[i], i)
        for k in range(4):
            same(ens_got[i][k], want_ens[k], (i, k))
