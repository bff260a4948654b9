"""fp32 prefill over V rows of very large and very small magnitude: the weighted sums on the way to an output stay within
the largest sum that probabilities of at most one give, so an output that fits fp32 comes out finite, and the probability
at a row's maximum is one, so small V rows keep their bits."""
import numpy as np
import pytest
import torch

from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("step", [2.0, 5.4, 30.0])
def test_outputs_that_fit_are_finite(d, step):
    """Scores rise by `step` (natural units) every 16 keys.  At most 64 keys of magnitude 3e36 with weights up to one sum to
    less than 2e38."""
    print("case:", d, step, flush=True)
    T = 64
    a = lambda x: np.asarray(x, np.int32)
    ctx = B.Context(0)
    plan = B.Plan(ctx, a([0, 1]), a([0]), a([T]), a([-1]), a([-1]), T, 1, 1, d, B.SP_F32)
    q, k, v = (np.zeros((T, 1, d), np.float32) for _ in range(3))
    q[:, 0, 0] = 1.0
    k[:, 0, 0] = step * (np.arange(T) // 16)
    v[:] = np.float32(3e36)
    v[:, 0, 1::2] *= -1
    O = torch.full((T, 1, d), 7.0, device="cuda")
    ctx.sp_forkjoin_prefill(plan, dev(q), dev(k), dev(v), O, 1.0)
    torch.cuda.synchronize()
    # every V row is the same, so every output is that row; 64 weights and their sum, each rounded to 2^-24
    np.testing.assert_allclose(O.cpu().numpy(), v, rtol=64 * 2.0 ** -24)
    plan.close()
    ctx.close()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("magnitude", [1e-36, 1.0, 1e35])
def test_error_does_not_depend_on_the_magnitude(d, magnitude):
    """Random scores of a few units.  At most 64 products of probabilities in (0, 1] and V, fp32: the error stays below
    what chains of 16 roundings and the exponential of one ulp give, 4e-7 of the norm, from 1e-36 up."""
    print("case:", d, magnitude, flush=True)
    T = 64
    a = lambda x: np.asarray(x, np.int32)
    ctx = B.Context(0)
    plan = B.Plan(ctx, a([0, 1]), a([0]), a([T]), a([-1]), a([-1]), T, 2, 2, d, B.SP_F32)
    rng = np.random.default_rng(d)
    q, k, v = (rng.standard_normal((T, 2, d), dtype=np.float32) for _ in range(3))
    v = (v * np.float32(magnitude)).astype(np.float32)
    O = torch.full((T, 2, d), 7.0, device="cuda")
    ctx.sp_forkjoin_prefill(plan, dev(q), dev(k), dev(v), O, 0.1)
    torch.cuda.synchronize()
    ref = orc.forkjoin_prefill(q, k, v, a([0, 1]), a([0]), a([T]), a([-1]), 0.1)
    got = O.cpu().numpy().astype(np.float64)
    assert np.linalg.norm((got - ref) / magnitude) <= 4e-7 * np.linalg.norm(ref / magnitude)
    plan.close()
    ctx.close()
