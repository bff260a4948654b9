"""How a prompt's keys are cut into pieces depends on the whole call: a prompt alone, in a batch, with more room in the
response cache or with its length on the host may round differently.  Each of them is the same attention to within
the rounding of its sums."""
import math

import numpy as np
import pytest
import torch

import sp_synth
from paper_2404_06910_amd import binding as B

from gpu_util import TORCH_DT, dev, make_plan

pytestmark = pytest.mark.gpu

D, LEN = 128, 30


def _one(ctx, dtype, Hq, Hkv, x, n, cap, on_host):
    """The first of n prompts (the others are copies of the second), LEN response rows in a cache of cap rows."""
    st = sp_synth.forkjoin_segtable(96, [[160, 200, 180]] * n, 24)
    T1 = st.n_tokens // n
    rep = lambda a: torch.cat([a[0]] + [a[1]] * (n - 1))
    plan = make_plan(ctx, st, Hq, Hkv, D, dtype)
    K, V = rep(x["k"]), rep(x["v"])
    assert K.shape[0] == n * T1
    Kr, Vr = (torch.zeros((n, cap, Hkv, D), dtype=K.dtype, device="cuda") for _ in range(2))
    Kr[:, :LEN], Vr[:, :LEN] = x["kr"], x["vr"]
    q, kn, vn = (x[i].expand(n, -1, -1).contiguous() for i in ("q", "kn", "vn"))
    o = torch.zeros_like(q)
    kept = dev(np.asarray([[2, 0]] * n, np.int32))
    kw = dict(resp_len_add=LEN) if on_host else dict(resp_len=dev(np.full(n, LEN, np.int32)))
    ctx.sp_pruned_decode(plan, kept, 2, K, V, Kr, Vr, cap, q, kn, vn, o, 1 / math.sqrt(D), **kw)
    torch.cuda.synchronize()
    plan.close()
    return o[0].float().cpu().numpy()


# dtype, what one call may differ from another by, relative to the output's largest value: fp32 sums of ~550 terms in
# another order (each step a rounding of 2^-24 of a sum of at most the largest value), rounded to bf16 (2^-8) where stored so
@pytest.mark.parametrize("dtype,tol", [("f32", 550 * 2.0 ** -24), ("bf16", 2.0 ** -8 + 550 * 2.0 ** -24)])
@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (8, 2)])
def test_the_same_prompt_in_other_calls(dtype, tol, Hq, Hkv):
    print("case:", dtype, Hq, Hkv, flush=True)
    ctx = B.Context(0)
    rng = np.random.default_rng(Hkv)
    f = lambda *s: torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).to(TORCH_DT[dtype]).cuda()
    T1 = sp_synth.forkjoin_segtable(96, [[160, 200, 180]], 24).n_tokens
    x = dict(k=[f(T1, Hkv, D), f(T1, Hkv, D)], v=[f(T1, Hkv, D), f(T1, Hkv, D)], kr=f(LEN, Hkv, D), vr=f(LEN, Hkv, D),
             q=f(1, Hq, D), kn=f(1, Hkv, D), vn=f(1, Hkv, D))
    want = _one(ctx, dtype, Hq, Hkv, x, 1, LEN + 1, True)
    for n, cap, on_host in ((1, LEN + 1, False), (1, 1000, False), (1, 1000, True), (3, LEN + 1, True), (80, LEN + 1, False)):
        got = _one(ctx, dtype, Hq, Hkv, x, n, cap, on_host)
        assert np.abs(got - want).max() <= tol * np.abs(want).max(), (n, cap, on_host)
        assert np.array_equal(got, _one(ctx, dtype, Hq, Hkv, x, n, cap, on_host))        # equal calls: equal bits
    ctx.close()
