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


def test_prompts_of_very_different_path_counts():
    """One prompt of 64 paths among many of one: the tables do not take a place for 64 paths of every prompt, and the look-up
    without such places finds the same keys (300 prompts: a launch that is small enough for the other one)."""
    n, d = 300, 64
    counts = [1] * n
    counts[7] = 64
    rng = np.random.default_rng(5)
    st = sp_synth.forkjoin_segtable(5, [[int(x) for x in rng.integers(1, 5, c)] for c in counts], 2)
    f = lambda *s: sp_synth.round_to_dtype(rng.standard_normal(s, dtype=np.float32), "f32")
    K, V, Kr, Vr = f(st.n_tokens, 2, d), f(st.n_tokens, 2, d), f(n, 1, 2, d), f(n, 1, 2, d)
    q, kn, vn = f(n, 2, d), f(n, 2, d), f(n, 2, d)
    kept = np.stack([[0, 1, -1] if c == 1 else [63, 5, 0] for c in counts]).astype(np.int32)   # path 1 only where there is one
    ctx = B.Context(0)
    plan = make_plan(ctx, st, 2, 2, d, "f32")
    o = torch.zeros((n, 2, d), device="cuda")
    ctx.sp_pruned_decode(plan, dev(kept), 3, dev(K), dev(V), dev(Kr), dev(Vr), 1, dev(q), dev(kn), dev(vn), o, 0.125)
    torch.cuda.synchronize()
    for b in (0, 6, 7, 8, n - 1):
        mine = [int(x) for x in kept[b] if 0 <= x < counts[b]]
        at = orc.joined_cache_index(st.prompt_seg_off, st.seg_tok_start, st.seg_tok_len, st.seg_path, b, mine)
        check_attn(o[b].cpu().numpy(), orc.pruned_decode_step(q[b], kn[b], vn[b], K, V, at, Kr[b, :0], Vr[b, :0], 0.125), "f32")
    plan.close()
    n = 40000
    seg = lambda first, second: np.concatenate([np.stack([np.full(n, first), np.full(n, second)], 1).ravel(), np.full(63, second)])
    off = np.append(np.arange(0, 2 * n, 2), 2 * n + 63).astype(np.int32)      # the last prompt has 64 paths
    parent = np.stack([np.full(n, -1), np.arange(n) * 2], 1).ravel()
    parent, path = np.concatenate([parent, np.full(63, 2 * n - 2)]), seg(-1, 0)
    path[2 * n:] = np.arange(1, 64)
    free = torch.cuda.mem_get_info()[0]
    plan = B.Plan(ctx, off, np.arange(2 * n + 63), np.ones(2 * n + 63), parent, path, 2 * n + 63, 1, 1, 64, B.SP_F32)
    took = free - torch.cuda.mem_get_info()[0]
    assert took < 16 << 20, took              # 32-byte items, 16-byte descriptors and a few numbers per prompt; 49 MB with places
    plan.close()
    ctx.close()
