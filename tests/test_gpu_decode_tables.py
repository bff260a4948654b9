"""Decode over kept tables at the edges of the two ways to look them up: prompts of different path counts up to 64 and
beyond, kept lists that fit a wave's lanes and longer ones, entries that name no path of their prompt."""
import math

import numpy as np
import pytest
import torch

import sp_synth
from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import check_attn, dev, make_plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv", [("bf16", 8, 2), ("bf16", 2, 2), ("f32", 4, 2)])
@pytest.mark.parametrize("counts", [(1, 3, 64), (1, 65, 3), (5, 1, 2)])
@pytest.mark.parametrize("k", [3, 63, 64])
def test_kept_tables(dtype, Hq, Hkv, counts, k):
    print("case:", dtype, Hq, Hkv, counts, k, flush=True)
    d, n = 64, len(counts)
    rng = np.random.default_rng(k + counts[1])
    st = sp_synth.forkjoin_segtable(9, [[int(x) for x in rng.integers(1, 9, c)] for c in counts], 3)
    f = lambda *s: sp_synth.round_to_dtype(rng.standard_normal(s, dtype=np.float32), dtype)
    K, V, Kr, Vr = f(st.n_tokens, Hkv, d), f(st.n_tokens, Hkv, d), f(n, 4, Hkv, d), f(n, 4, Hkv, d)
    q, kn, vn = f(n, Hq, d), f(n, Hkv, d), f(n, Hkv, d)
    kept = np.full((n, k), -1, np.int32)
    for b, c in enumerate(counts):
        some = rng.permutation(c)[:max(1, min(c, k) - 1)]
        kept[b, rng.permutation(k)[:len(some)]] = some
        free = np.flatnonzero(kept[b] < 0)
        if len(free):
            kept[b, free[-1]] = [c, 64, 2 ** 31 - 1][b]               # no path of this prompt
    ctx = B.Context(0)
    plan = make_plan(ctx, st, Hq, Hkv, d, dtype)
    o = torch.zeros((n, Hq, d), dtype=dev(q, dtype).dtype, device="cuda")
    scale = 1 / math.sqrt(d)
    ctx.sp_pruned_decode(plan, dev(kept), k, dev(K, dtype), dev(V, dtype), dev(Kr, dtype), dev(Vr, dtype), 4, dev(q, dtype),
                         dev(kn, dtype), dev(vn, dtype), o, scale, resp_len_add=2)
    torch.cuda.synchronize()
    for b, c in enumerate(counts):
        mine = [int(x) for x in kept[b] if 0 <= x < c]
        at = orc.joined_cache_index(st.prompt_seg_off, st.seg_tok_start, st.seg_tok_len, st.seg_path, b, mine)
        ref = orc.pruned_decode_step(q[b], kn[b], vn[b], K, V, at, Kr[b, :2], Vr[b, :2], scale)
        check_attn(o[b].float().cpu().numpy(), ref, dtype, "prompt %d" % b)
    plan.close()
    ctx.close()
