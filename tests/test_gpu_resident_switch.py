"""Launches of many steps against launches of one step on the same handle type, bit for bit:
every tiling and scheme option of the on-chip steps, with the on-chip path switched on and off
(needs an MI355X)."""
import numpy as np
import pytest

import synth
from tests.test_gpu_parity import hx  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu

BOOKS = ("t", "stored", "rain", "outflow", "clamp", "steps", "dt_min", "dt_max_seen")
OPTIONS = ["plain", "masked", "viscous", "flux", "dirichlet", "infiltration", "soil"]


def scene(nq, nr, option, seed=5, **kw):
    """A wet, flowing slope; masked, viscous, flux and dirichlet: the parallelogram's corners cut
    off, with an open rim, and a column of boundary cells."""
    sc = synth.c1_planar(nq, nr, t_end=1e9)
    h, v1, v2 = synth.random_state(sc, seed)
    rng = np.random.default_rng(seed)
    kw = dict(h0=h, v10=v1, v20=v2, z=sc.z + 0.05 * rng.random(sc.n), **kw)
    if option == "infiltration":
        kw.update(f_inf=1e-5, h_inf=0.01)
    if option == "soil":
        kw.update(alpha_s=0.005 + 0.005 * rng.random(sc.n))
    if option in ("masked", "viscous", "flux", "dirichlet"):
        q = np.arange(nq)[None, :] + 0.5 * np.arange(nr)[:, None]
        act = (q >= min(nr // 2, nq // 3)).astype(np.uint8)
        if option != "masked" and nq > 3:
            act[:, -1] = 2 if option == "dirichlet" else 3
        m = act.reshape(-1) > 0
        kw.update(active=act.reshape(-1), mask_code=synth.OUTFLOW, h0=h * m, v10=v1 * m,
                  v20=v2 * m, visc=option == "viscous")
    return sc.with_(**kw)


def same(a, b, what):
    for f in a[0]:
        assert np.array_equal(a[0][f], b[0][f], equal_nan=True), (what, f)
    for f in BOOKS:
        assert a[1][f] == b[1][f], (what, f, a[1][f], b[1][f])


# one raster for every tiling (tile variant, stacked tiles) that the on-chip steps are built
# for, each with a ragged last workgroup; a device has 256 compute units
TILINGS = [(200, 19, 0, 1), (64, 1029, 0, 2), (130, 1100, 0, 4), (64, 40, 1, 1),
           (250, 530, 1, 2), (450, 1003, 1, 4), (90, 50, 2, 1), (300, 1100, 2, 2),
           (1000, 1000, 2, 4)]


@pytest.mark.parametrize("option", OPTIONS)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nq,nr,tile,sub", TILINGS)
def test_many_steps_a_launch_equal_single_launches(hx, nq, nr, tile, sub, precision, option):
    sc = scene(nq, nr, option)
    print(f"[on-chip {nq}x{nr} tile {tile} x {sub} {precision} {option}]", flush=True)
    out = []
    for on in (True, False):
        sim = hx.Sim.from_scenario(sc, precision, tile=tile)
        sim.set_resident(on)
        for n in (113, 40):  # two launches of up to 100 steps; then from the other buffer
            sim.run(1e9, max_steps=n)
        out.append((sim.state_numpy(), sim.books()))
        # FP64 viscous cells in stacks too large for a thread's registers stay with single
        # steps, and so do masked FP64 rasters in stacks of four (slower on chip)
        built = not (precision == "fp64" and
                     ((option == "viscous" and tile == 2) or
                      (option in ("masked", "viscous", "flux", "dirichlet") and tile > 0 and
                       sub == 4)))
        assert (sim.resident_launches() > 0) == (on and built)
        del sim
    same(out[0], out[1], (nq, nr, tile, sub))


@pytest.mark.parametrize("option", ["plain", "masked", "viscous", "flux", "dirichlet"])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("tile,scale", [(0, 1), (0, 5), (0, 9), (2, 1)])
def test_ensemble_groups_equal_single_launches(hx, tile, scale, precision, option):
    """Scenarios of one, several and ragged tiles; scale 5 and 9: stacks of two and four."""
    sizes = [(1, 1), (64, 16), (65, 17), (130, 40), (30, 100), (200, 13)]
    scs = [scene(nq, nr * scale, option, seed=k) for k, (nq, nr) in enumerate(sizes)]
    ends = [1.0 + 0.3 * k for k in range(len(scs))]
    out = []
    for on in (True, False):
        ens = hx.Ensemble.from_scenarios(scs, precision, mode="batched", tile=tile)
        ens.set_resident(on)
        ens.run(ends)
        ens.run(1e9, max_steps=110)  # more steps than one launch takes
        out.append([(ens.state_numpy(k), ens.books(k)) for k in range(len(scs))])
        built = not (option == "viscous" and precision == "fp64" and tile == 2)
        assert (ens.resident_launches() > 0) == (on and built)
        del ens
    for k in range(len(scs)):
        print(f"[ensemble tile {tile} scale {scale} {precision} {option} {k}]", flush=True)
        same(out[0][k], out[1][k], k)


@pytest.mark.parametrize("on", [True, False])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_run_shape_does_not_change_results(hx, precision, on):
    """Graphs (or launches) of odd and even lengths, graphs longer than the step ring, and runs
    cut into uneven pieces with kernel timings in between, all against single launches."""
    sc = synth.catchment(72, 64, 2.0, config=2, t_end=80.0)
    ref = hx.Sim.from_scenario(sc, precision)
    ref.set_resident(False)
    ref.run(sc.t_end)
    want = ref.state_numpy(), ref.books()
    assert want[1]["steps"] > 300
    for spg in (1, 3, 7, 8, 300):
        sim = hx.Sim.from_scenario(sc, precision, steps_per_graph=spg)
        sim.set_resident(on)
        sim.run(sc.t_end)
        same((sim.state_numpy(), sim.books()), want, spg)
    sim = hx.Sim.from_scenario(sc, precision, steps_per_graph=16)
    sim.set_resident(on)
    done = 0
    for piece in (1, 13, 2, 29, 200):
        sim.run(sc.t_end, max_steps=piece)
        done += piece
        assert sim.books()["steps"] == done
        sim.time_kernel(5)
    sim.run(sc.t_end)
    same((sim.state_numpy(), sim.books()), want, "pieces")
    assert (sim.resident_launches() > 0) == on


# (raster, precision, option, steps of a run): a run goes on chip only where that is faster
ROUTES = [
    ((64, 64), "fp32", "plain", 1, True),
    ((64, 64), "fp64", "viscous", 1, True),
    ((300, 300), "fp32", "plain", 1, False),      # two tiles a workgroup: set up for one step
    ((300, 300), "fp64", "plain", 3, False),
    ((300, 300), "fp64", "plain", 4, True),
    ((512, 512), "fp64", "viscous", 15, False),
    ((512, 512), "fp64", "viscous", 16, True),
    ((1000, 1000), "fp32", "plain", 7, False),
    ((1000, 1000), "fp32", "plain", 8, True),
    ((1000, 1000), "fp32", "masked", 8, False),
    ((1000, 1000), "fp32", "masked", 16, True),
    ((2000, 260), "fp32", "viscous", 200, False),  # idle compute units
    ((1000, 1000), "fp64", "plain", 15, False),
    ((1000, 1000), "fp64", "infiltration", 16, True),
    ((1000, 1000), "fp64", "masked", 200, False),
    ((750, 750), "fp64", "plain", 200, False),
    ((500, 600), "fp64", "flux", 200, False),
]


@pytest.mark.parametrize("size,precision,option,steps,on_chip", ROUTES)
def test_runs_take_the_faster_path(hx, size, precision, option, steps, on_chip):
    print(f"[route {size} {precision} {option} {steps} steps]", flush=True)
    sim = hx.Sim.from_scenario(scene(*size, option), precision)
    sim.run(1e9, max_steps=steps)
    assert sim.books()["steps"] == steps
    assert (sim.resident_launches() > 0) == on_chip


def test_switch_arguments(hx):
    L = hx.lib()
    assert L.hexsv_sim_set_resident(None, 1) == hx.EINVAL
    assert L.hexsv_ensemble_set_resident(None, 1) == hx.EINVAL
    assert L.hexsv_sim_resident_launches(None) == -1
    assert L.hexsv_ensemble_resident_launches(None) == -1
    sim = hx.Sim.from_scenario(scene(8, 8, "plain"), "fp64")
    assert L.hexsv_sim_set_resident(sim._h, 2) == hx.EINVAL
