"""sp_pruned_decode where the key lists are long enough to be cut into pieces, and the grouped-head kernel: against the
oracle, at key counts on and around the piece and tile boundaries, with every head grouping the dispatch knows; and the
scratch regions of the pieces: streams do not share one."""
import math

import numpy as np
import pytest
import torch

import sp_synth
from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import TORCH_DT, attn_tol, dev, make_plan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def _setup(ctx, rng, dtype, Hq, Hkv, d, st, k, resp, bias, cap=None):
    f = lambda *s: sp_synth.round_to_dtype(rng.standard_normal(s, dtype=np.float32), dtype)
    Bn, cap = st.n_prompts, cap or max(resp) + 1
    x = dict(kp=f(st.n_tokens, Hkv, d), vp=f(st.n_tokens, Hkv, d), kr=f(Bn, cap, Hkv, d), vr=f(Bn, cap, Hkv, d),
             q=f(Bn, Hq, d), kn=f(Bn, Hkv, d), vn=f(Bn, Hkv, d))
    x["kept"] = np.stack([rng.permutation(int(st.path_off[b + 1] - st.path_off[b]))[:k] for b in range(Bn)]).astype(np.int32)
    x["pos"] = x["slopes"] = x["pos_resp"] = x["new_pos"] = None
    if bias:
        x["pos"] = rng.uniform(0, 300, st.n_tokens).astype(np.float32)
        x["slopes"] = sp_synth.geometric_slopes(Hq)
        x["pos_resp"] = rng.uniform(300, 400, (Bn, cap)).astype(np.float32)
        x["new_pos"] = np.full(Bn, 401, np.float32)
    x["plan"] = make_plan(ctx, st, Hq, Hkv, d, dtype, x["pos"], x["slopes"])
    x["dev"] = {n: dev(x[n], dtype) for n in ("kp", "vp", "kr", "vr", "q", "kn", "vn")}
    x["dev"]["kept"] = dev(x["kept"])
    x["dev"]["resp_len"] = dev(np.asarray(resp, np.int32))
    for n in ("pos_resp", "new_pos"):
        x["dev"][n] = None if x[n] is None else dev(x[n])
    x["k"], x["cap"], x["scale"] = k, cap, 1 / math.sqrt(d)
    return x


def _decode(ctx, x, dtype, o=None):
    t = x["dev"]
    if o is None:
        o = torch.full(t["q"].shape, float("nan"), dtype=TORCH_DT[dtype], device="cuda")
    ctx.sp_pruned_decode(x["plan"], t["kept"], x["k"], t["kp"], t["vp"], t["kr"], t["vr"], x["cap"], t["q"], t["kn"],
                         t["vn"], o, x["scale"], resp_len=t["resp_len"], pos_resp=t["pos_resp"], new_pos=t["new_pos"])
    return o


def _check(got, x, st, resp, dtype):
    mx, mean = attn_tol(dtype)
    for b in range(st.n_prompts):
        idx = orc.joined_cache_index(st.prompt_seg_off, st.seg_tok_start, st.seg_tok_len, st.seg_path, b, x["kept"][b])
        n = resp[b]
        kw = {} if x["pos"] is None else dict(pos_prefill=x["pos"], pos_resp=x["pos_resp"][b, :n], pos_new=x["new_pos"][b],
                                              alibi_slopes=x["slopes"])
        ref = orc.pruned_decode_step(x["q"][b], x["kn"][b], x["vn"][b], x["kp"], x["vp"], idx, x["kr"][b, :n],
                                     x["vr"][b, :n], x["scale"], **kw)
        err = np.abs(got[b].astype(np.float64) - ref)
        assert err.max() <= mx and err.mean() <= mean, "prompt %d: max %.3e mean %.3e" % (b, err.max(), err.mean())


# dtype, Hq, Hkv, d, preamble, document lengths, query length, kept paths, response lengths, bias
CASES = [
    ("bf16", 4, 4, 128, 64, [[200, 190, 33], [60, 1, 64]], 24, 2, [0, 130], False),   # one-head kernel, up to 7 pieces
    ("bf16", 4, 4, 64, 31, [[200, 190]], 9, 2, [77], True),
    ("bf16", 4, 2, 128, 96, [[96, 95, 97]], 1, 2, [0], False),                        # 2 heads; 290 keys: 3 pieces + 1
    ("bf16", 4, 2, 64, 95, [[50, 45]], 0, 2, [1], True),                              # 192 keys: exactly 2 pieces
    ("bf16", 6, 2, 128, 40, [[300, 280]], 5, 2, [63], False),                         # 3 heads padded to 4
    ("bf16", 8, 2, 128, 96, [[160, 200, 180, 220, 90]] * 3, 24, 4, [0, 15, 120], True),
    ("bf16", 5, 1, 64, 17, [[120, 130]], 7, 1, [3], True),                            # 5 heads padded to 8
    ("bf16", 16, 2, 128, 64, [[150, 170]], 11, 2, [16], False),                       # 8 heads
    ("bf16", 12, 1, 64, 64, [[150, 170], [16, 15]], 11, 2, [16, 0], False),           # 12 heads: 8 + 4
    ("bf16", 8, 2, 128, 1, [[1, 1]], 1, 1, [0], False),                               # 3 keys, all in the short path
    ("f32", 8, 2, 128, 64, [[100, 90]], 3, 2, [40], True),                            # 4 heads fp32, 8 pieces
    ("f32", 2, 2, 64, 64, [[100, 90]], 3, 2, [90], False),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "%s-h%d/%d-d%d-P%d-k%d%s" % (c[0], c[1], c[2], c[3], c[4], c[7], "-b" if c[9] else ""))
def test_pieces_match_the_oracle(ctx, case):
    dtype, Hq, Hkv, d, P, lens, Lq, k, resp, bias = case
    print("case:", case, flush=True)
    rng = np.random.default_rng(CASES.index(case))
    st = sp_synth.forkjoin_segtable(P, lens, max(Lq, 1), "grouped" if bias else "interleaved")
    x = _setup(ctx, rng, dtype, Hq, Hkv, d, st, k, resp, bias)
    got = _decode(ctx, x, dtype)
    again = _decode(ctx, x, dtype)
    torch.cuda.synchronize()
    assert torch.equal(got, again)                       # the counters are back at zero, the merge order is fixed
    _check(got.float().cpu().numpy(), x, st, resp, dtype)


@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (4, 1)])
def test_more_ranges_than_a_wave_has_lanes(ctx, Hq, Hkv):
    """A kept path of 100 segments that lie apart in the token pool: keys behind the 64th range."""
    rng = np.random.default_rng(8)
    n = 100
    lens = rng.integers(1, 9, n)
    start = np.cumsum(np.concatenate([[5], lens + 2]))[:n]
    i32 = lambda a: np.asarray(a, np.int32)
    seg_start, seg_len = i32(np.concatenate([[0], start])), i32(np.concatenate([[3], lens]))
    T, d = int(seg_start[-1] + seg_len[-1]), 128
    st = sp_synth.SegTable(1, T, i32([0, n + 1]), seg_start, seg_len, i32(range(-1, n)), i32([-1] + [0] * n), i32([0, 1]),
                           None, None, None)
    x = _setup(ctx, rng, "bf16", Hq, Hkv, d, st, 1, [9], False)
    got = _decode(ctx, x, "bf16")
    torch.cuda.synchronize()
    _check(got.float().cpu().numpy(), x, st, [9], "bf16")


def test_streams_have_their_own_scratch():
    """One plan, 20 streams: overlapping launches on all of them give what a lone launch gives, bit for bit, and so do
    launches on the per-thread stream."""
    print("case: decode on 20 streams of one plan", flush=True)
    ctx = B.Context(0)
    rng = np.random.default_rng(4)
    st = sp_synth.forkjoin_segtable(96, [[160, 200, 180, 220]] * 2, 24)
    xs = [_setup(ctx, rng, "bf16", 8, 2, 128, st, 3, [20, 90], False) for _ in range(20)]
    want = []
    for x in xs:
        x["plan"] = xs[0]["plan"]
        want.append(_decode(ctx, x, "bf16"))
        torch.cuda.synchronize()
    got = [torch.full_like(w, float("nan")) for w in want]
    streams = [torch.cuda.Stream() for _ in xs]
    torch.cuda.synchronize()
    for _ in range(3):
        for x, o, s in zip(xs, got, streams):
            ctx.sp_set_stream(s.cuda_stream)
            _decode(ctx, x, "bf16", o)
    torch.cuda.synchronize()
    for w, o in zip(want, got):
        assert torch.equal(w, o)
    ctx.sp_set_stream(2)                                 # hipStreamPerThread
    for x, w in zip(xs[:3], want):
        o = torch.full_like(w, float("nan"))
        torch.cuda.synchronize()
        _decode(ctx, x, "bf16", o)
        torch.cuda.synchronize()
        assert torch.equal(w, o)
    ctx.close()
