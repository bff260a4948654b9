"""fp32 prefill where its 16-row waves and 16-key steps can go wrong: row counts around the tile sizes, every head
grouping, steps that straddle ancestor ranges, and rows whose step holds keys they do not see."""
import math

import numpy as np
import pytest
import torch

from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu

# fp32 sums of D products and of at most ~700 probabilities in chains of 8 to 16, each rounded to 2^-24 of values of
# magnitude <= 8, and a hardware exp2 of one ulp: well under 2e-5 of outputs of magnitude ~1.
TOL = 2e-5


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def _chain_and_leaves(chain, leaves, gap):
    """root -> chain of segments lying apart -> leaves; returns table arrays and the token count."""
    start, length, parent, path, tok = [], [], [], [], 0
    for i, n in enumerate(chain):
        start.append(tok); length.append(n); parent.append(i - 1); path.append(-1); tok += n + gap
    for j, n in enumerate(leaves):
        start.append(tok); length.append(n); parent.append(len(chain) - 1); path.append(j); tok += n + gap
    a = lambda x: np.asarray(x, np.int32)
    return (a([0, len(start)]), a(start), a(length), a(parent), a(path)), tok


def _run(ctx, args, T, q, k, v, pos=None, slopes=None, head_major=False):
    plan = B.Plan(ctx, *args, T, q.shape[1], k.shape[1], q.shape[2], B.SP_F32, tok_pos=pos, alibi_slopes=slopes)
    Q, K, V = dev(q), dev(k), dev(v)
    if head_major:
        K, V = (x.transpose(0, 1).contiguous().transpose(0, 1) for x in (K, V))
    O = torch.full_like(Q, 7.0)
    ctx.sp_forkjoin_prefill(plan, Q, K, V, O, 1.0 / math.sqrt(q.shape[2]))
    torch.cuda.synchronize()
    return O.cpu().numpy()


@pytest.mark.parametrize("Hq,Hkv,d,chain,bias,head_major", [
    (2, 2, 128, [1], False, False), (4, 4, 64, [16], True, True), (4, 2, 128, [15, 3], True, False),
    (6, 3, 64, [17, 40, 1], False, True), (8, 2, 128, [33, 16, 5, 9], False, False), (8, 1, 64, [130], True, False),
    (12, 4, 128, [20, 7] * 6, True, True),
])
def test_rows_around_the_tile_sizes(ctx, Hq, Hkv, d, chain, bias, head_major):
    leaves = [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 97]
    args, T = _chain_and_leaves(chain, leaves, gap=3)
    print("case:", Hq, Hkv, d, chain, bias, head_major, flush=True)
    rng = np.random.default_rng(d + len(chain))
    q, k, v = (rng.standard_normal((T, h, d), dtype=np.float32) for h in (Hq, Hkv, Hkv))
    pos = rng.uniform(0, 200, T).astype(np.float32) if bias else None
    slopes = np.exp2(-np.arange(1, Hq + 1)).astype(np.float32) if bias else None
    got = _run(ctx, args, T, q, k, v, pos, slopes, head_major)
    ref = orc.forkjoin_prefill(q, k, v, *args[:4], 1.0 / math.sqrt(d), tok_pos=pos, alibi_slopes=slopes)
    out = np.isnan(ref)
    assert np.all(got[out] == 7.0)                         # rows of no segment are left alone
    assert np.abs(got[~out] - ref[~out]).max() <= TOL


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_values_behind_a_row_do_not_reach_it(ctx, bad):
    """Rows 0..39 of a 60-row run are checked with K and V of rows 40..59 not finite; rows from 40 on see them."""
    args, T = _chain_and_leaves([9], [60], gap=2)
    rng = np.random.default_rng(3)
    q, k, v = (rng.standard_normal((T, h, 64), dtype=np.float32) for h in (4, 2, 2))
    ref = orc.forkjoin_prefill(q, k, v, *args[:4], 0.125)
    first = int(args[1][1]) + 40
    k2, v2 = k.copy(), v.copy()
    v2[first:first + 20] = bad
    k2[first + 1:first + 20] = bad
    print("case: bad", bad, flush=True)
    got = _run(ctx, args, T, q, k2, v2)
    seen = ~np.isnan(ref)
    seen[first:] = False
    assert np.abs(got[seen] - ref[seen]).max() <= TOL
    assert not np.isfinite(got[first:first + 20]).any()
