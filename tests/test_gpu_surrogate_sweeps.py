"""Surrogate kernels whose workgroups sweep several tiles or rows (needs an MI355X)."""
import numpy as np
import pytest
import torch

from oracle import surrogate as so
from tests.test_gpu_parity import hx  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def rel_l2(a, b):
    return float((a - b).norm() / b.norm().clamp_min(1e-30))


# 512 workgroups compute the weight gradients: one tile each at most, exactly one, and
# several with a remainder (tiles are 64 x 4 cells; 8 samples of 72, 64 and 130 tiles)
@pytest.mark.parametrize("nq,nr", [(1, 1), (130, 95), (64, 256), (321, 102)])
def test_batch_gradient_is_the_mean_of_its_samples(hx, nq, nr):
    """With a power of two of samples the loss gradient's bfloat16 rounding scales exactly, so
    the batch's gradient is the mean of the samples' up to FP32 summation: about 1e5 terms in
    blocks of at most 2048, each rounded to 6e-8, well inside 2e-5."""
    batch = 8
    rng = np.random.default_rng(31)
    p = (so.init_params(31, 4, 32, out_scale=1.0)
         + rng.normal(scale=0.02, size=so.num_params(4, 32))).astype(np.float32)
    f = torch.from_numpy(rng.normal(size=(batch, nq * nr, so.FEATURES)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.normal(size=(batch, nq * nr, 3)).astype(np.float32)).cuda()
    sur = hx.Surrogate(4, 32)
    sur.set_params(p)
    loss, g = sur.gradient(f, t, nq, nr)
    one = [sur.gradient(f[b].contiguous(), t[b].contiguous(), nq, nr) for b in range(batch)]
    mean = torch.stack([x[1].double() for x in one]).mean(0)
    e = rel_l2(g.double(), mean)
    print(f"[surrogate batch gradient {nq}x{nr}] rel L2 {e:.2e}", flush=True)
    assert e <= 2e-5
    assert loss == pytest.approx(sum(x[0] for x in one) / batch, rel=1e-9)
    again = sur.gradient(f, t, nq, nr)
    assert torch.equal(again[1], g) and again[0] == loss  # a fixed order of summation
