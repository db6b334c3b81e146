"""How a surrogate call runs its network: as a sweep, by tiles or layer by layer, whichever is
fastest for the samples, with the same outputs bit for bit (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle.surrogate as so
import synth
from tests.test_gpu_parity import hx  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


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


# (samples, raster, mask, a forward's route, a forced one-kernel forward's, a gradient's)
CALLS = [
    (1, 100, 75, False, "sweep", "sweep", "sweep"),
    (1, 100, 75, True, "sweep", "sweep", "chain"),   # masked activations are not kept on the way
    (16, 128, 120, False, "sweep", "sweep", "sweep"),
    (2, 512, 512, True, "sweep", "sweep", "chain"),
    (64, 58, 58, True, "sweep", "sweep", "chain"),
    (512, 16, 16, False, "tiles", "tiles", "sweep"),  # a sweep would be mostly margins
    (512, 16, 16, True, "tiles", "tiles", "chain"),
    (8, 3, 1000, True, "tiles", "tiles", "chain"),
    (4096, 8, 8, False, "chain", "tiles", "chain"),
    (4096, 1, 1, False, "chain", "sweep", "chain"),
    (64, 128, 128, True, "chain", "sweep", "chain"),
    (8, 60, 1000, True, "chain", "tiles", "chain"),
]


@pytest.mark.parametrize("batch,nq,nr,masked,forward,forced,gradient", CALLS)
def test_calls_take_the_fastest_route(hx, batch, nq, nr, masked, forward, forced, gradient):
    print(f"[route {batch}x{nq}x{nr} masked {masked}]", flush=True)
    sur, grid, f, t = network(hx, batch, nq, nr, masked)
    shape = (batch, nq, nr, grid)
    assert sur.route(*shape) == forward and sur.route(*shape, "gradient") == gradient
    o, (loss, g) = sur.forward(f, nq, nr, grid), sur.gradient(f, t, nq, nr, grid)
    for on in (True, False):
        sur.set_fused(on)
        assert sur.route(*shape) == (forced if on else "chain")
        assert sur.route(*shape, "gradient") == (gradient if on else "chain")
        assert torch.equal(sur.forward(f, nq, nr, grid)[:, :3], o[:, :3])
        loss1, g1 = sur.gradient(f, t, nq, nr, grid)
        assert loss1 == loss and torch.equal(g1, g)


# parts of a tile, whole ones, and remainders in either direction, with every kind of border;
# as many samples as it takes for a forced one-kernel forward to choose the tiles
TILED = [(b, k) for k in ("walls", "masked", "periodic", "periodic masked")
         for b in [(512, 5, 6), (512, 16, 16), (512, 14, 30), (1500, 15, 13)] +
         ([(560, 17, 9), (512, 20, 16)] if "masked" in k else [])]


@pytest.mark.parametrize("size,kind", TILED)
def test_tiles_equal_the_chain(hx, size, kind):
    batch, nq, nr = size
    print(f"[tiles {batch}x{nq}x{nr} {kind}]", flush=True)
    sur, _, f, _ = network(hx, batch, nq, nr, False, seed=nq)
    rng = np.random.default_rng(nr)
    active = None
    if "masked" in kind:
        active = (rng.random((nr, nq)) < 0.7).astype(np.uint8)
        active[0, 0], active[-1, -1] = 1, 0
    side = (hx.PERIODIC if "periodic" in kind else hx.WALL,) * 4
    grid = hx.Grid(nq, nr, 1.0, side=side, active=active)
    sur.set_fused(True)
    assert sur.route(batch, nq, nr, grid) == "tiles"
    out = sur.forward(f, nq, nr, grid)
    sur.set_fused(False)
    assert torch.equal(sur.forward(f, nq, nr, grid)[:, :3], out[:, :3])


def test_noalloc_takes_the_tiles(hx):
    batch, nq, nr = 512, 16, 16
    sur, _, f, _ = network(hx, batch, nq, nr, False)
    want = sur.forward(f, nq, nr)
    out = torch.full((batch * nq * nr, 4), 7.0, device="cuda")
    assert sur.route(batch, nq, nr) == "tiles"
    sur.forward_noalloc(f, nq, nr, out)
    assert torch.equal(out[:, :3], want[:, :3]) and bool((out[:, 3] == 7).all())


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

    hx._check(hx.lib().hexsv_surrogate_forward(sur._h, None, 1, nq, nr, hx._ptr(f), hx._ptr(out),
                                               hx._stream()))
    assert torch.equal(out.view(-1, 4)[:, :3], want[:, :3])
    assert bool((buf[:shift] == 7).all()) and bool((buf[shift + 4 * nq * nr:] == 7).all())


@pytest.mark.parametrize("batch,nq,nr,masked,shift", [
    (512, 16, 16, False, 0), (4096, 8, 8, False, 0), (64, 128, 128, True, 0), (1, 100, 75, False, 0),
    (512, 16, 16, False, 1), (1, 100, 75, True, 3)])
def test_a_captured_forward_needs_no_workspace(hx, batch, nq, nr, masked, shift):
    """Capture as the first call of a surrogate; later calls move its workspace."""
    print(f"[capture {batch}x{nq}x{nr} masked {masked} shift {shift}]", flush=True)
    sur, grid, f, _ = network(hx, batch, nq, nr, masked)
    other, _, f2, _ = network(hx, batch, nq, nr, masked)
    x = f.clone()
    buf = torch.full((4 * batch * nq * nr + 8,), 7.0, device="cuda")
    out = buf[shift:shift + 4 * batch * nq * nr]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        hx._check(hx.lib().hexsv_surrogate_forward(sur._h, grid._h if grid else None, batch, nq, nr,
                                                   hx._ptr(x), hx._ptr(out), hx._stream()))
    for k in range(3):
        x.copy_((f if k != 1 else -f2))
        buf.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        want = other.forward(x, nq, nr, grid)
        assert torch.equal(out.view(-1, 4)[:, :3], want[:, :3]), k
        assert bool((buf[:shift] == 7).all()) and bool((buf[shift + out.numel():] == 7).all())
        many = batch * (k + 2)  # a workspace of another size, at another address
        sur.set_fused(False)
        sur.forward(torch.zeros((many * nq * nr, so.FEATURES), device="cuda"), nq, nr, grid)
        sur.set_fused(True)


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


@pytest.mark.parametrize("nq,nr,masked,way", [
    (100, 75, False, "sweep"), (512, 512, False, "sweep"), (60, 1000, True, "chain"),
    (512, 512, True, "chain")])
def test_windows_take_the_fastest_route(hx, nq, nr, masked, way):
    sc, sim, sur = still(hx, nq, nr, masked)
    assert sur.route(1, nq, nr, sim.grid, "window") == way
    windows(sc, sim, sur)
    got = sim.state_numpy()
    assert hx.lib().hexsv_sim_window_kernels(sim._h) == (8 if way == "chain" else 6)
    for on in (True, False):
        sur.set_fused(on)
        windows(sc, sim, sur)
        again = sim.state_numpy()
        assert all(np.array_equal(got[k], again[k]) for k in got)


def test_windows_follow_set_fused(hx):
    """The windows' graphs are captured on the first call; set_fused afterwards holds for them."""
    sc, sim, sur = still(hx, 100, 75, False)
    assert hx.lib().hexsv_sim_window_kernels(sim._h) == 0
    windows(sc, sim, sur)
    for on in (False, True, False):
        sur.set_fused(on)
        windows(sc, sim, sur)
        assert hx.lib().hexsv_sim_window_kernels(sim._h) == (6 if on else 8)


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


def test_route_arguments(hx):
    L = hx.lib()
    sur = hx.Surrogate(4, 32)
    for args in ((None, None, 1, 8, 8, 0), (sur._h, None, 0, 8, 8, 0), (sur._h, None, 1, 8, 8, 3)):
        assert L.hexsv_surrogate_route(*args) == hx.EINVAL
    assert L.hexsv_sim_window_kernels(None) == hx.EINVAL
    assert hx.Surrogate(3, 32).route(16, 512, 512) == "chain"
