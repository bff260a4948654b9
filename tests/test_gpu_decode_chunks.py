"""sp_pruned_decode where the query heads of a KV head are more than one workgroup takes: every chunk reads the same K and V
rows, and only such calls read them through the caches; the workgroups of (prompt, KV head) pairs that divide by 8 are put
in another order."""
import numpy as np
import pytest
import torch

import sp_synth
from paper_2404_06910_amd import binding as B

from test_gpu_decode_pieces import _check, _decode, _setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hq,Hkv", [("f32", 6, 2), ("f32", 5, 1), ("f32", 12, 2), ("f32", 8, 1), ("f32", 10, 1), ("f32", 4, 2),
                                          ("bf16", 9, 1), ("bf16", 16, 1), ("bf16", 34, 2)])
@pytest.mark.parametrize("d,prompts,bias", [(64, 2, False), (128, 3, True), (128, 8, False), (64, 16, True)])
def test_chunks_match_the_oracle(dtype, Hq, Hkv, d, prompts, bias):
    print("case:", dtype, Hq, Hkv, d, prompts, bias, flush=True)
    ctx = B.Context(0)
    rng = np.random.default_rng(Hq + d)
    st = sp_synth.forkjoin_segtable(40, ([[90, 61, 130], [33, 1, 64], [200, 7, 5]] * 6)[:prompts], 9)
    resp = ([17, 0, 40] * 6)[:prompts]
    x = _setup(ctx, rng, dtype, Hq, Hkv, d, st, 2, resp, bias)
    got = _decode(ctx, x, dtype)
    torch.cuda.synchronize()
    _check(got.float().cpu().numpy(), x, st, resp, dtype)
    x["plan"].close()
    ctx.close()
