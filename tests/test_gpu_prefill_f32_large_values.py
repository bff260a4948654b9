"""fp32 prefill over V rows of large magnitude: the weighted sums on the way to an output stay within the largest sum that
probabilities of at most one give, so an output that fits fp32 comes out finite."""
import numpy as np
import pytest
import torch

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
