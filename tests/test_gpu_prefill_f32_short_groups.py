"""fp32 prefill of short row groups, where the plan takes tiles of 16 or 32 rows: parity at the sizes around the tiles, and no
launch of far more waves than have rows."""
import math

import numpy as np
import pytest
import torch

import sp_synth
from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import check_attn, dev, make_plan, run_prefill
from hip_graphs import Graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,d", [(3, 3, 64), (4, 2, 128), (8, 2, 64)])
@pytest.mark.parametrize("pre,docs,q", [(1, [1, 1, 1], 1), (16, [5, 9, 11, 2], 3), (64, [13] * 6, 4), (17, [28, 28, 25], 4),
                                        (70, [33, 47, 20, 1], 15), (5, [1, 100, 2, 3], 2)])
def test_short_groups_match_the_oracle(Hq, Hkv, d, pre, docs, q):
    print("case:", Hq, Hkv, d, pre, docs, q, flush=True)
    ctx = B.Context(0)
    rng = np.random.default_rng(pre + d)
    for packing in ("interleaved", "grouped"):               # documents and queries in one row group, and apart
        st = sp_synth.forkjoin_segtable(pre, [docs, docs[::-1]], q, packing)
        qq, k, v = (rng.standard_normal((st.n_tokens, h, d), dtype=np.float32) for h in (Hq, Hkv, Hkv))
        got, plan = run_prefill(ctx, st, qq, k, v, "f32")
        ref = orc.forkjoin_prefill(qq, k, v, st.prompt_seg_off, st.seg_tok_start, st.seg_tok_len, st.seg_parent,
                                   1.0 / math.sqrt(d))
        check_attn(got, ref, "f32")
        plan.close()
    ctx.close()


@pytest.mark.parametrize("Hq,Hkv", [(32, 32), (32, 16), (32, 8)])
@pytest.mark.parametrize("doc,q", [(1, 1), (5, 3), (24, 4)])
def test_launched_waves_have_rows(Hq, Hkv, doc, q):
    """At most half as many again as there are 16-row blocks, and one round of the slots."""
    ctx = B.Context(0)
    n = 400
    st = sp_synth.forkjoin_segtable(64, [[doc] * n], q)
    plan = make_plan(ctx, st, Hq, Hkv, 64, "f32")
    Q, K = (torch.zeros((st.n_tokens, h, 64), device="cuda") for h in (Hq, Hkv))
    V, O = torch.zeros_like(K), torch.zeros_like(Q)
    stream = torch.cuda.Stream()

    def work():
        ctx.sp_set_stream(stream.cuda_stream)
        ctx.sp_forkjoin_prefill(plan, Q, K, V, O, 0.125)
    g = Graph(stream, work)
    blocks = (4 + n * -(-(doc + q) // 16)) * Hq
    (grid,) = g.grids()
    assert blocks <= grid[0] <= 1.5 * blocks + 8 * 1024, (grid, blocks)
    g.destroy()
    plan.close()
    ctx.close()
