"""Saliency at the row lengths where the last vectors of a row change form: one to four vectors a lane, a wave with fewer than
the waves before it, and calls of so many rows that the last vectors go one after the other."""
import numpy as np
import pytest
import torch

import sp_synth
from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,vecs,tail", [(5, v, 1) for v in (0, 1, 63, 64, 65, 255, 256, 257, 319, 449, 512, 513, 577, 768,
                                                                769, 961, 1023, 1024, 1025, 1279, 2047)] +
                         [(4096, 257, 0), (4097, 1, 0), (4097, 257, 3), (4097, 1025, 1)])
def test_row_lengths(dtype, rows, vecs, tail):
    print("case:", dtype, rows, vecs, tail, flush=True)
    per = 4 if dtype == "f32" else 8
    vocab = vecs * per + tail
    rng = np.random.default_rng(vecs)
    x = sp_synth.round_to_dtype(rng.normal(0, 3, (rows, vocab)).astype(np.float32), dtype)
    target = rng.integers(0, vocab, rows).astype(np.int32)
    row_path = np.arange(rows, dtype=np.int32) // 8
    n_slots = int(row_path[-1]) + 1
    full = torch.full((rows, (vocab + per - 1) // per * per), 50.0)           # what lies behind a row's end is not read
    full[:, :vocab] = torch.from_numpy(x)
    ctx = B.Context(0)
    score = torch.full((n_slots,), float("nan"), device="cuda")
    ctx.sp_path_saliency(dev(full.numpy(), dtype)[:, :vocab], dev(target), dev(row_path), n_slots, score)
    torch.cuda.synchronize()
    # a row's lp is a few fp32 roundings of a logsumexp below 32 in magnitude, and a slot has at most 8 rows
    ref = orc.path_saliency(x, target, row_path, n_slots)
    assert np.abs(score.cpu().numpy() - ref).max() <= 8 * 4 * 32 * 2.0 ** -24
    ctx.close()
