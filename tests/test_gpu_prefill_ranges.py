"""bf16 prefill behind several ancestor ranges: stages that end inside a range, reach into the next one or into the own
run, or hold three ranges and more, at the range counts where the search in LDS changes over (8 are kept there)."""
import math

import numpy as np
import pytest
import torch

import sp_synth
from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import check_attn, dev
from test_gpu_prefill_f32_tiles import _chain_and_leaves

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,d", [(2, 2, 128), (4, 2, 64), (8, 2, 128)])
@pytest.mark.parametrize("chain", [[31, 1], [64, 32], [7, 9, 11, 5, 100, 3, 33], [20] * 6 + [70, 21], [64] * 8, [40] * 9,
                                   [1] * 8])
@pytest.mark.parametrize("bias", [False, True])
def test_stages_across_ranges(Hq, Hkv, d, chain, bias):
    print("case:", Hq, Hkv, d, chain, bias, flush=True)
    args, T = _chain_and_leaves(chain, [1, 33, 90], gap=3)
    rng = np.random.default_rng(len(chain) + Hq)
    q, k, v = (sp_synth.round_to_dtype(rng.standard_normal((T, h, d), dtype=np.float32), "bf16") for h in (Hq, Hkv, Hkv))
    pos = rng.uniform(0, 200, T).astype(np.float32) if bias else None
    slopes = np.exp2(-np.arange(1, Hq + 1)).astype(np.float32) if bias else None
    ctx = B.Context(0)
    plan = B.Plan(ctx, *args, T, Hq, Hkv, d, B.SP_BF16, tok_pos=pos, alibi_slopes=slopes)
    Q = dev(q, "bf16")
    O = torch.full_like(Q, 7.0)
    scale = 1.0 / math.sqrt(d)
    ctx.sp_forkjoin_prefill(plan, Q, dev(k, "bf16"), dev(v, "bf16"), O, scale)
    torch.cuda.synchronize()
    ref = orc.forkjoin_prefill(q, k, v, *args[:4], scale, tok_pos=pos, alibi_slopes=slopes)
    got = O.float().cpu().numpy()
    check_attn(got, ref, "bf16", str(chain))
    assert np.all(got[np.isnan(ref)] == 7.0)
    plan.close()
    ctx.close()
