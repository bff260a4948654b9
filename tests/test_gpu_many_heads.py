"""Prefill with more KV heads than a signed 16-bit number holds (a work item packs the query and the KV head in 32 bits)."""
import math
import types

import numpy as np
import pytest
import torch

from paper_2404_06910_amd import binding as B

from fullsize_oracle import oracle_by_segment
from gpu_util import SP_DT, TORCH_DT, check_attn
from wide_plans import chain_table

pytestmark = pytest.mark.gpu

SMALL = dict(prompts=1, chain=[19], docs=[5, 40], query=3)
WIDE = dict(prompts=1, chain=[224], docs=[1] * 32, cached_chain=True)


@pytest.mark.parametrize("dtype,d,H,kw", [("bf16", 128, 40000, SMALL), ("bf16", 64, 65535, SMALL), ("f32", 64, 40000, SMALL),
                                          ("bf16", 128, 33000, WIDE)], ids=["bf16", "bf16_64", "f32", "wide"])
def test_many_kv_heads(dtype, d, H, kw):
    args, T, cached = chain_table(**kw)
    print("case:", dtype, d, H, T, flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(H)
    Q, K, V = (torch.randn((T, H, d), generator=g, device="cuda", dtype=TORCH_DT[dtype]) for _ in range(3))
    O = torch.zeros_like(Q)
    ctx = B.Context(0)
    plan = B.Plan(ctx, *args, T, H, H, d, SP_DT[dtype], seg_cached=cached)
    assert (len(plan.work_items()[1]) - 1 == 256) == (kw is WIDE)
    scale = 1.0 / math.sqrt(d)
    ctx.sp_forkjoin_prefill(plan, Q, K, V, O, scale)
    torch.cuda.synchronize()
    heads = [0, 32767, 32768, H - 1]
    st = types.SimpleNamespace(prompt_seg_off=args[0], seg_tok_start=args[1], seg_tok_len=args[2], seg_parent=args[3])
    q, k, v, o = (t[:, heads].float().cpu().numpy() for t in (Q, K, V, O))
    toks, ref = oracle_by_segment(st, q, k, v, scale, 0, list(range(len(heads))))
    if cached is not None:
        ref[toks < 224] = np.nan
    check_attn(o[toks], ref, dtype, "heads %s" % heads)
    plan.close()
    ctx.close()
