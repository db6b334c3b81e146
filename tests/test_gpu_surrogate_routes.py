"""Which kernels a surrogate call launches: the one-launch network or the layer chain, whichever
is faster for the samples, with the same outputs bit for bit (needs an MI355X)."""
import numpy as np
import pytest
import torch
from torch.profiler import ProfilerActivity, profile

import oracle.surrogate as so
import synth
from tests.test_gpu_parity import hx  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def kernels(call):
    """Names of the kernels that call() launches, from graphs too, in a Counter-like dict."""
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    count = {}
    for e in p.events():
        for k in ("k_hexnet4", "k_hexconv<", "k_win_apply", "k_win_last", "k_win_probe"):
            if k in e.name:
                count[k] = count.get(k, 0) + 1
    return count


def network(hx, batch, nq, nr, masked, seed=3):
    rng = np.random.default_rng(seed)
    p = (so.init_params(6, 4, 32, out_scale=1.0)
         + rng.normal(scale=0.05, size=so.num_params(4, 32))).astype(np.float32)
    sur = hx.Surrogate(4, 32)
    sur.set_params(p)
    grid = None
    if masked:
        active = (rng.random((nr, nq)) < 0.8).astype(np.uint8)
        active[0, 0] = 1
        active[-1, -1] = 0
        grid = hx.Grid(nq, nr, 1.0, side=(hx.WALL,) * 4, active=active)
    n = batch * nq * nr
    f = torch.from_numpy(rng.normal(size=(n, so.FEATURES)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.normal(size=(n, 3)).astype(np.float32)).cuda()
    return sur, grid, f, t


# (samples, raster, mask, one launch for a forward, for a gradient)
CALLS = [
    (1, 100, 75, False, True, True),
    (1, 100, 75, True, True, False),
    (16, 128, 120, False, True, True),
    (512, 16, 16, False, True, True),
    (4096, 8, 8, False, False, False),   # mostly margins
    (4096, 1, 1, False, False, False),
    (512, 16, 16, True, False, False),
    (64, 64, 64, True, False, False),    # two strips for 64 columns, with predicates
    (8, 60, 1000, True, False, False),
    (2, 512, 512, True, True, False),    # activations to keep as well
]


@pytest.mark.parametrize("batch,nq,nr,masked,forward,gradient", CALLS)
def test_calls_take_the_faster_route(hx, batch, nq, nr, masked, forward, gradient):
    print(f"[route {batch}x{nq}x{nr} masked {masked}]", flush=True)
    sur, grid, f, t = network(hx, batch, nq, nr, masked)
    out = {}
    seen = kernels(lambda: out.update(o=sur.forward(f, nq, nr, grid)))
    assert (seen.get("k_hexnet4", 0), seen.get("k_hexconv<", 0)) == ((1, 0) if forward else (0, 4))
    seen = kernels(lambda: out.update(g=sur.gradient(f, t, nq, nr, grid)))
    assert (seen.get("k_hexnet4", 0), seen.get("k_hexconv<", 0)) == ((1, 0) if gradient else (0, 4))
    for on in (True, False):
        sur.set_fused(on)
        assert torch.equal(sur.forward(f, nq, nr, grid)[:, :3], out["o"][:, :3])
        loss, g = sur.gradient(f, t, nq, nr, grid)
        assert loss == out["g"][0] and torch.equal(g, out["g"][1])


@pytest.mark.parametrize("shift", [0, 1, 2, 3, 4])
def test_forward_to_any_float_address(hx, shift):
    """Outputs that are no multiple of 16 bytes: the four floats of a cell are one store only
    where they are."""
    nq, nr = 100, 75
    sur, _, f, _ = network(hx, 1, nq, nr, False)
    want = sur.forward(f, nq, nr)
    buf = torch.full((4 * nq * nr + 8,), 7.0, device="cuda")
    out = buf[shift:shift + 4 * nq * nr]
    assert (out.data_ptr() % 16 == 0) == (shift % 4 == 0)

    def call():
        hx._check(hx.lib().hexsv_surrogate_forward(sur._h, None, 1, nq, nr, hx._ptr(f),
                                                   hx._ptr(out), hx._stream()))

    call()
    assert torch.equal(out.view(-1, 4)[:, :3], want[:, :3])
    assert bool((buf[:shift] == 7).all()) and bool((buf[shift + 4 * nq * nr:] == 7).all())
    # the general route: packed input, the workspace's output, a copy
    seen = kernels(call)
    assert seen == {"k_hexnet4": 1}
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    assert any("k_pack_features" in e.name for e in p.events()) == (shift % 4 != 0)


def still(hx, nq, nr, masked):
    """Still water in a closed basin: a network of zeros is kept in every window."""
    sc = synth.c1_planar(nq, nr, t_end=1e9)
    z = np.zeros(sc.n)
    act = None
    if masked:
        act = np.ones((nr, nq), np.uint8)
        act[:, : nq // 8] = 0
    h = np.full(sc.n, 0.05) * (1 if act is None else act.reshape(-1))
    sc = sc.with_(z=z, h0=h, v10=z, v20=z, i_a=0.0, side=(synth.WALL,) * 4, active=act,
                  mask_code=synth.WALL)
    sur = hx.Surrogate(4, 32)
    sur.set_params(np.zeros(sur.num_params, np.float32))
    sur.set_scales([0.05, 0.01, 1.0, 0.001, 0.001, 0.05])
    return sc, hx.Sim.from_scenario(sc, "fp32"), sur


def windows(sc, sim, sur, n=16):
    sim.set_state(sc.h0, sc.v10, sc.v20, 0.0)
    kept = sim.run_surrogate(sur, float(n), 1.0, 16, residual_tol=float("inf"))
    assert kept == (n, 0)


@pytest.mark.parametrize("nq,nr,masked,fused", [(100, 75, False, True), (512, 512, False, True),
                                                (60, 1000, True, False)])
def test_windows_take_the_faster_route(hx, nq, nr, masked, fused):
    sc, sim, sur = still(hx, nq, nr, masked)
    seen = kernels(lambda: windows(sc, sim, sur))
    assert seen["k_win_probe"] == 16
    assert (seen.get("k_hexnet4", 0), seen.get("k_win_last", 0)) == ((16, 0) if fused else (0, 16))


def test_windows_follow_set_fused(hx):
    """The windows' graphs are captured on the first call; set_fused afterwards holds for them."""
    sc, sim, sur = still(hx, 100, 75, False)
    windows(sc, sim, sur)
    for on in (False, True, False):
        sur.set_fused(on)
        seen = kernels(lambda: windows(sc, sim, sur))
        got = tuple(seen.get(k, 0) for k in ("k_hexnet4", "k_win_apply", "k_hexconv<", "k_win_last"))
        assert got == ((16, 16, 0, 0) if on else (0, 0, 48, 16))


def test_a_new_surrogate_at_an_old_address(hx):
    """A simulation that captured windows with a surrogate since destroyed uses the next one's
    weights and buffers, also where the allocator hands its address out again."""
    sc, sim, sur = still(hx, 100, 75, False)
    windows(sc, sim, sur)
    old, kept = sur._h.value, []
    del sur
    for _ in range(16):
        kept.append(hx.Surrogate(4, 32))
        if kept[-1]._h.value == old:
            break
    sur = kept[-1]
    p = np.zeros(sur.num_params, np.float32)
    p[-3:] = 0.01, 0.002, -0.001  # the last layer's biases: a constant change per window
    sur.set_params(p)
    sur.set_scales([0.05, 0.01, 1.0, 0.001, 0.001, 0.05])
    windows(sc, sim, sur)
    got = sim.state_numpy()
    fresh = hx.Sim.from_scenario(sc, "fp32")
    windows(sc, fresh, sur)
    want = fresh.state_numpy()
    assert not np.array_equal(want["h"], sc.h0.astype(np.float32))
    for k in want:
        assert np.array_equal(got[k], want[k]), k
