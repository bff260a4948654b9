"""sp_pruned_decode over cached V rows that hold infinities: a lane that has no key of its own must add nothing, whatever
the row it reads in its place holds."""
import math

import numpy as np
import pytest
import torch

import sp_synth
from paper_2404_06910_amd import binding as B

from gpu_util import TORCH_DT, make_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv,d", [("bf16", 8, 2, 128), ("bf16", 4, 2, 64), ("bf16", 2, 2, 64), ("bf16", 2, 2, 128),
                                            ("bf16", 16, 2, 64), ("f32", 4, 2, 64), ("f32", 2, 2, 128)])
@pytest.mark.parametrize("doc", [24, 200, 312])
def test_infinite_values_stay_infinite(dtype, Hq, Hkv, d, doc):
    """Key j has +inf in dim j % d: every dim of the output is a positive weight times +inf plus finite terms.  The
    documents give 113, 289 and 401 keys: one to four pieces, several of them ending in the middle of a step."""
    print("case:", dtype, Hq, Hkv, d, doc, flush=True)
    ctx = B.Context(0)
    st = sp_synth.forkjoin_segtable(64, [[doc]], 24)
    rng = np.random.default_rng(doc)
    T = st.n_tokens
    f = lambda *s: torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).to(TORCH_DT[dtype]).cuda()
    plan = make_plan(ctx, st, Hq, Hkv, d, dtype)
    K, V, q, kn, vn = f(T, Hkv, d), f(T, Hkv, d), f(1, Hq, d), f(1, Hkv, d), f(1, Hkv, d)
    j = torch.arange(T, device="cuda")
    V[j, :, j % d] = float("inf")
    vn[0, :, 5] = float("inf")
    Kr, Vr = torch.zeros((1, 2, Hkv, d), dtype=K.dtype, device="cuda"), torch.zeros((1, 2, Hkv, d), dtype=K.dtype, device="cuda")
    o = torch.zeros_like(q)
    kept = torch.zeros((1, 1), dtype=torch.int32, device="cuda")
    ctx.sp_pruned_decode(plan, kept, 1, K, V, Kr, Vr, 2, q, kn, vn, o, 1 / math.sqrt(d))
    torch.cuda.synchronize()
    want = torch.zeros(d, dtype=torch.bool, device="cuda")
    want[j % d] = True
    want[5] = True
    assert torch.equal(torch.isposinf(o[0]), want.expand(Hq, d)), o[0, 0]
    assert not torch.isnan(o).any()
    plan.close()
    ctx.close()
