"""The wide bf16 prefill against the oracle and, for all heads and rows, against the other bf16 kernel, which takes each
prompt of the same call by itself (too little work for the wide one)."""
import math
import types

import numpy as np
import pytest
import torch

import sp_synth
from paper_2404_06910_amd import binding as B

from fullsize_oracle import oracle_by_segment
from gpu_util import check_attn
from wide_plans import CASES, chain_table

pytestmark = pytest.mark.gpu


def _plan(ctx, args, T, Hq, Hkv, cached, **kw):
    return B.Plan(ctx, *args, T, Hq, Hkv, 128, B.SP_BF16, seg_cached=cached, **kw)


def _one_prompt(args, cached, b):
    off, start, length, parent, path = args
    s = slice(int(off[b]), int(off[b + 1]))
    par = np.where(parent[s] >= 0, parent[s] - off[b], -1).astype(np.int32)
    return (np.asarray([0, s.stop - s.start], np.int32), start[s], length[s], par, path[s]), \
        None if cached is None else cached[s]


def _inputs(T, Hq, Hkv, head_major, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    normal = lambda *s: torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16)
    kv = (lambda: normal(Hkv, T, 128).transpose(0, 1)) if head_major else (lambda: normal(T, Hkv, 128))
    return normal(T, Hq, 128), kv(), kv()


@pytest.mark.parametrize("bias", [False, True])
@pytest.mark.parametrize("name", sorted(CASES))
def test_wide_prefill(name, bias):
    Hq, Hkv, kw = CASES[name]
    args, T, cached = chain_table(**kw)
    print("case:", name, bias, "tokens", T, flush=True)
    Q, K, V = _inputs(T, Hq, Hkv, head_major=bias, seed=len(name))
    rng = np.random.default_rng(len(name))
    extra = {}
    if bias:
        extra = dict(tok_pos=rng.uniform(0, 900, T).astype(np.float32),
                     alibi_slopes=np.exp2(-np.linspace(1, 8, Hq)).astype(np.float32))
    ctx = B.Context(0)
    plan = _plan(ctx, args, T, Hq, Hkv, cached, **extra)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert len(plan.work_items()[1]) - 1 == (n_cu + 7) // 8 * 8      # the wide kernel
    scale = 1.0 / math.sqrt(128)
    O, O2 = torch.full_like(Q, 7.0), torch.full_like(Q, 7.0)
    ctx.sp_forkjoin_prefill(plan, Q, K, V, O, scale)
    for b in range(kw["prompts"]):
        one, one_cached = _one_prompt(args, cached, b)
        p = _plan(ctx, one, T, Hq, Hkv, one_cached, **extra)
        assert len(p.work_items()[1]) - 1 > (n_cu + 7) // 8 * 8
        ctx.sp_forkjoin_prefill(p, Q, K, V, O2, scale)
        p.close()
    torch.cuda.synchronize()
    assert torch.equal(O == 7.0, O2 == 7.0)                          # the same rows, and no others, are written
    a, c = O.float(), O2.float()
    assert torch.isfinite(a).all()
    # Each side rounds its weights to 8 bits (2^-9 of a weight; the weights sum to 1, so 2^-9 of the largest value at most)
    # and its result (2^-9 of that).
    bound = 2.0 ** -8 * (c.abs() + V.float().abs().max())
    worst = ((a - c).abs() / bound).max().item()
    assert worst <= 1.0 and (a - c).norm().item() <= 1e-2 * c.norm().item(), worst
    st = types.SimpleNamespace(prompt_seg_off=args[0], seg_tok_start=args[1], seg_tok_len=args[2], seg_parent=args[3])
    heads = [0, Hq - 1]
    q, k, v = Q.float().cpu().numpy(), K.float().cpu().numpy(), V.float().cpu().numpy()
    b = kw["prompts"] - 1
    toks, ref = oracle_by_segment(st, q, k, v, scale, b, heads, extra.get("tok_pos"), extra.get("alibi_slopes"))
    if cached is not None:
        for s in range(int(args[0][b]), int(args[0][b + 1])):
            if cached[s]:
                ref[(toks >= args[1][s]) & (toks < args[1][s] + args[2][s])] = np.nan
    check_attn(a.cpu().numpy()[toks][:, heads], ref, "bf16", name)
    plan.close()
    ctx.close()


def test_infinite_values_of_a_path_stay_in_it():
    """Paths that share a tile: values of one that are not finite leave no trace in the others."""
    Hq, Hkv, kw = CASES["siblings"]
    args, T, _ = chain_table(**kw)
    Q, K, V = _inputs(T, Hq, Hkv, False, 3)
    ctx = B.Context(0)
    plan = _plan(ctx, args, T, Hq, Hkv, None)
    O, O2 = torch.zeros_like(Q), torch.zeros_like(Q)
    ctx.sp_forkjoin_prefill(plan, Q, K, V, O, 0.09)
    off, start, length, parent, path = args
    sick = torch.zeros(T, dtype=torch.bool, device="cuda")
    for s in range(len(start)):
        if path[s] >= 0 and path[s] % 3 == 1:
            sick[int(start[s]):int(start[s] + length[s])] = True
    K[sick], V[sick] = float("nan"), float("inf")
    ctx.sp_forkjoin_prefill(plan, Q, K, V, O2, 0.09)
    torch.cuda.synchronize()
    assert torch.equal(O[~sick], O2[~sick]) and not torch.isfinite(O2[sick]).any()
    plan.close()
    ctx.close()


def test_wide_prefill_replayed():
    """Captured and replayed, with other inputs and eager launches between: nothing of a launch is left in the next."""
    Hq, Hkv, kw = CASES["ragged"]
    args, T, _ = chain_table(**kw)
    ctx = B.Context(0)
    plan = _plan(ctx, args, T, Hq, Hkv, None)
    Q, K, V = _inputs(T, Hq, Hkv, False, 4)
    O, O2 = torch.zeros_like(Q), torch.zeros_like(Q)
    ctx.sp_forkjoin_prefill(plan, Q, K, V, O2, 0.09)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.sp_set_stream(torch.cuda.current_stream().cuda_stream)
        ctx.sp_forkjoin_prefill(plan, Q, K, V, O, 0.09)
    ctx.sp_set_stream(torch.cuda.current_stream().cuda_stream)
    for i in range(3):
        Q.copy_(Q.roll(1, 0))
        graph.replay()
        ctx.sp_forkjoin_prefill(plan, Q, K, V, O2, 0.09)
        torch.cuda.synchronize()
        assert torch.equal(O, O2), i
    plan.close()
    ctx.close()
