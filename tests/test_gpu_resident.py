"""Resident steps (many steps of a raster that fits on the chip in one launch) against the
batched ensemble's single-step launches with the same tile, bit for bit, and against the FP64
oracle (needs an MI355X)."""
import numpy as np
import pytest

import oracle
import synth
from tests.test_gpu_parity import hx  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

STEPS = 37


def scene(nq, nr, option, seed=5):
    """A wet, flowing slope; masked: the parallelogram's corners cut off, with an open rim."""
    sc = synth.c1_planar(nq, nr, t_end=1e9)
    h, v1, v2 = synth.random_state(sc, seed)
    kw = dict(h0=h, v10=v1, v20=v2, z=sc.z + 0.05 * np.random.default_rng(seed).random(sc.n))
    if option != "plain":
        q = np.arange(nq)[None, :] + 0.5 * np.arange(nr)[:, None]
        act = (q >= min(nr // 2, nq // 3)).astype(np.uint8)
        if option == "viscous" and nq > 3:
            act[:, -1] = 3  # a column of given-flux cells
        m = act.reshape(-1) > 0
        kw.update(active=act.reshape(-1), mask_code=synth.OUTFLOW, h0=h * m, v10=v1 * m,
                  v20=v2 * m, visc=option == "viscous")
    return sc.with_(**kw)


# one tile; a second one of one column or row; workgroups of one, two and four stacked tiles
# (variant v's rows are 4, 8 and 16 high; a device has 256 compute units), each with a ragged
# last workgroup
SHAPES = [(1, 1, 0), (64, 4, 0), (65, 5, 0), (200, 19, 0), (64, 1029, 0), (130, 700, 0),
          (64, 40, 1), (250, 530, 1), (130, 1500, 1), (90, 50, 2), (500, 600, 2), (520, 1004, 2)]


@pytest.mark.parametrize("option", ["plain", "masked", "viscous"])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nq,nr,tile", SHAPES)
def test_resident_equals_single_launches(hx, nq, nr, tile, precision, option):
    sc = scene(nq, nr, option)
    print(f"[resident {nq}x{nr} tile {tile} {precision} {option}]", flush=True)
    sim = hx.Sim.from_scenario(sc, precision, tile=tile)
    ens = hx.Ensemble.from_scenarios([sc], precision, mode="batched", tile=tile)
    for n in (STEPS, 3):  # the second run starts from the other buffer
        sim.run(1e9, max_steps=n)
        ens.run(1e9, max_steps=n)
    a, b = sim.state_numpy(), ens.state_numpy(0)
    for k in a:
        assert np.array_equal(a[k], b[k], equal_nan=True), k
    x, y = sim.books(), ens.books(0)
    for k in ("t", "stored", "rain", "outflow", "clamp", "steps", "dt_min", "dt_max_seen"):
        assert x[k] == y[k], (k, x[k], y[k])


@pytest.mark.parametrize("nq,nr,tile", [(65, 5, 0), (130, 70, 1), (200, 90, 2)])
def test_resident_matches_the_oracle_to_the_end_time(hx, nq, nr, tile):
    """FP64 is the oracle's arithmetic operation for operation; the run ends at t_end exactly,
    in the middle of a launch."""
    sc = scene(nq, nr, "plain")
    G = oracle.grid(sc.nq, sc.nr, sc.a, sc.side, sc.segs, sc.active, sc.mask_code)
    p = oracle.params(sc.g, sc.cfl, sc.dt_max, sc.h_dry, sc.alpha_s)
    h, v1, v2, b, _ = oracle.run(G, sc.z, sc.theta, sc.alpha_p, p, oracle.rain(*sc.rain), sc.h0,
                                 sc.v10, sc.v20, 6.5)
    sim = hx.Sim.from_scenario(sc, "fp64", tile=tile, steps_per_graph=16).run(6.5)
    st, bk = sim.state_numpy(), sim.books()
    for k, ref in (("h", h), ("v1", v1), ("v2", v2)):
        assert np.array_equal(st[k], ref), k
    assert bk["t"] == 6.5 and bk["steps"] == b.steps
    assert bk["residual"] <= 1e-12


@pytest.mark.parametrize("option", ["plain", "masked", "viscous"])
@pytest.mark.parametrize("precision,tile", [("fp64", -1), ("fp32", -1), ("fp64", 0)])
def test_resident_ensemble_equals_single_runs(hx, precision, tile, option):
    """Scenarios of one, several and ragged tiles, stopped at their own end times and then
    resumed: every scenario as if it ran alone."""
    scs = [scene(nq, nr, option, seed=k) for k, (nq, nr) in
           enumerate([(1, 1), (64, 16), (65, 17), (130, 40), (30, 100), (200, 13)])]
    ens = hx.Ensemble.from_scenarios(scs, precision, mode="batched", tile=tile)
    used = ens.info()["tile"]
    ends = [1.0 + 0.7 * k for k in range(len(scs))]
    ens.run(ends)
    ens.run(1e9, max_steps=150)  # more steps than one launch takes
    for k, sc in enumerate(scs):
        print(f"[resident ensemble {option} {precision} tile {used} scenario {k}]", flush=True)
        sim = hx.Sim.from_scenario(sc, precision, tile=used)
        sim.run(ends[k])
        assert sim.books()["t"] == ends[k]
        sim.run(1e9, max_steps=150)
        a, b = ens.state_numpy(k), sim.state_numpy()
        for f in a:
            assert np.array_equal(a[f], b[f], equal_nan=True), f
        x, y = ens.books(k), sim.books()
        for f in ("t", "stored", "rain", "outflow", "clamp", "steps", "dt_min", "dt_max_seen"):
            assert x[f] == y[f], (f, x[f], y[f])
