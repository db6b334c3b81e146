"""The one-launch surrogate forward against the layer-by-layer one (needs an MI355X)."""
import numpy as np
import pytest
import torch

from oracle import surrogate as so
from tests.test_gpu_parity import hx  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


# strips are 58 columns wide; segments of one row, of several with a shorter last one, and
# whole strips (batch); rasters narrower than the taps' reach
@pytest.mark.parametrize("nq,nr,batch", [(1, 1, 1), (2, 3, 1), (57, 1, 2), (58, 8, 1), (59, 9, 3),
                                         (116, 75, 1), (117, 130, 2), (64, 300, 40), (9, 500, 300)])
@pytest.mark.parametrize("kind", ["plain", "masked", "periodic"])
def test_fused_forward_equals_the_layer_chain(hx, nq, nr, batch, kind):
    """The same products in the same order with the same roundings: equal bit for bit."""
    rng = np.random.default_rng(nq * 1000 + nr)
    p = (so.init_params(5, 4, 32, out_scale=1.0)
         + rng.normal(scale=0.05, size=so.num_params(4, 32))).astype(np.float32)
    grid = None
    if kind == "masked":
        active = (rng.random((nr, nq)) < 0.8).astype(np.uint8)
        active[0, 0] = 1
        grid = hx.Grid(nq, nr, 1.0, side=(hx.WALL,) * 4, active=active)
    elif kind == "periodic":
        grid = hx.Grid(nq, nr, 1.0, side=(hx.PERIODIC,) * 4)
    f = torch.from_numpy(rng.normal(size=(batch * nq * nr, so.FEATURES)).astype(np.float32)).cuda()
    sur = hx.Surrogate(4, 32)
    sur.set_params(p)
    one = sur.forward(f, nq, nr, grid=grid)
    sur.set_fused(False)
    chain = sur.forward(f, nq, nr, grid=grid)
    assert torch.equal(one[:, :3], chain[:, :3])  # the fourth float is no output
    if batch * nq * nr <= 262144:
        sur.set_fused(True)
        out = torch.full_like(chain, 7.0)
        sur.forward_noalloc(f, nq, nr, out, grid=grid)
        assert torch.equal(out[:, :3], chain[:, :3])
        assert bool((out[:, 3] == 7.0).all())


@pytest.mark.parametrize("nq,nr,batch", [(1, 1, 1), (59, 9, 3), (117, 130, 2)])
@pytest.mark.parametrize("kind", ["plain", "masked"])
def test_gradient_from_the_fused_forward(hx, nq, nr, batch, kind):
    """The fused forward leaves the gradient the chain's activations: equal bit for bit."""
    rng = np.random.default_rng(nq + nr)
    p = (so.init_params(6, 4, 32, out_scale=1.0)
         + rng.normal(scale=0.05, size=so.num_params(4, 32))).astype(np.float32)
    grid = None
    if kind == "masked":
        active = (rng.random((nr, nq)) < 0.8).astype(np.uint8)
        active[0, 0] = 1
        grid = hx.Grid(nq, nr, 1.0, side=(hx.WALL,) * 4, active=active)
    n = batch * nq * nr
    f = torch.from_numpy(rng.normal(size=(n, so.FEATURES)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.normal(size=(n, 3)).astype(np.float32)).cuda()
    sur = hx.Surrogate(4, 32)
    sur.set_params(p)
    loss, g = sur.gradient(f, t, nq, nr, grid)
    sur.set_fused(False)
    loss0, g0 = sur.gradient(f, t, nq, nr, grid)
    assert torch.equal(g, g0) and loss == loss0
