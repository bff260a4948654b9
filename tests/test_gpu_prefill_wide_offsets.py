"""The wide bf16 prefill at the ends of the addresses that are accepted: Q and O rows almost 2^26 elements apart (a lane's
offset inside a block of 32 rows has 32 bits and comes to 31 such strides), and tokens behind 4 GB of K and V in either layout."""
import math
import types

import numpy as np
import pytest
import torch

from paper_2404_06910_amd import binding as B

from fullsize_oracle import oracle_by_segment
from gpu_util import check_attn
from wide_plans import chain_table

pytestmark = pytest.mark.gpu


def _run(args, n_tokens, cached, H, Q, K, V, O):
    ctx = B.Context(0)
    plan = B.Plan(ctx, *args, n_tokens, H, H, 128, B.SP_BF16, seg_cached=cached)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert len(plan.work_items()[1]) - 1 == (n_cu + 7) // 8 * 8                # the wide kernel
    scale = 1.0 / math.sqrt(128)
    ctx.sp_forkjoin_prefill(plan, Q, K, V, O, scale)
    torch.cuda.synchronize()
    plan.close()
    ctx.close()
    return scale


def _normal(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)


def _table(args):
    return types.SimpleNamespace(prompt_seg_off=args[0], seg_tok_start=args[1], seg_tok_len=args[2], seg_parent=args[3])


@pytest.mark.parametrize("head_major", [False, True])
def test_tokens_behind_4GB(head_major):
    H, shift = 32, (1 << 19) + 4096
    args, T, _ = chain_table(prompts=8, chain=[600], docs=[128] * 12, query=24)
    print("case:", head_major, T + shift, flush=True)
    assert shift * H * 128 * 2 > 1 << 32

    def tensor(seed, by_head):
        t = torch.zeros((H, T + shift, 128) if by_head else (T + shift, H, 128), dtype=torch.bfloat16, device="cuda")
        t = t.transpose(0, 1) if by_head else t
        t[shift:] = _normal(seed, T, H, 128)
        return t

    Q, K, V = tensor(1, False), tensor(2, head_major), tensor(3, head_major)
    O = torch.zeros_like(Q)
    scale = _run((args[0], args[1] + np.int32(shift)) + args[2:], T + shift, None, H, Q, K, V, O)
    heads = [0, 13, 31]
    q, k, v, o = (t[shift:, heads].float().cpu().numpy() for t in (Q, K, V, O))
    for b in (0, 7):
        toks, ref = oracle_by_segment(_table(args), q, k, v, scale, b, [0, 1, 2])
        check_attn(o[toks], ref, "bf16")


def test_largest_query_stride():
    """Documents of blocks of 1 to 32 rows behind one cached chain, whose rows Q and O do not have (25 GB each as it is)."""
    H, stride, chain, docs = 64, (1 << 26) - 128, 16384, [64, 33, 40] + [1] * 24 + [20, 5]
    n = sum(docs)
    print("case:", n, flush=True)
    assert (31 * stride + 256) * 2 < 1 << 32
    i32 = lambda *a: np.asarray(a, np.int32)
    at = np.cumsum([0] + docs[:-1])
    m = len(docs)
    args = i32(0, m + 1), i32(n, *at), i32(chain, *docs), i32(-1, *[0] * m), i32(-1, *range(m))
    size = (n - 1) * stride + H * 128
    Q, O = (torch.as_strided(torch.empty(size, dtype=torch.bfloat16, device="cuda"), (n, H, 128), (stride, 128, 1)) for _ in range(2))
    Q.copy_(_normal(1, n, H, 128))
    O.zero_()
    K, V = _normal(2, n + chain, H, 128), _normal(3, n + chain, H, 128)
    scale = _run(args, n + chain, np.asarray([1] + [0] * m, np.uint8), H, Q, K, V, O)
    heads = [0, 40, 63]
    q, o = (t[:, heads].float().cpu().numpy() for t in (Q, O))
    k, v = (t[:, heads].double().cpu().numpy() for t in (K, V))
    for a, r in zip(at, docs):
        for h in range(3):
            s = q[a:a + r, h].astype(np.float64) @ np.concatenate([k[n:, h], k[a:a + r, h]]).T * scale
            s[:, chain:][np.triu_indices(r, 1)] = -np.inf
            p = np.exp(s - s.max(1, keepdims=True))
            ref = p @ np.concatenate([v[n:, h], v[a:a + r, h]]) / p.sum(1, keepdims=True)
            check_attn(o[a:a + r, h], ref, "bf16", "document at %d" % a)
