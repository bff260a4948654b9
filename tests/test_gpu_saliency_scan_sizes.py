"""The scan that sums a path's rows, at the sizes where it changes over to 1024 threads: against the oracle, and bit for bit
against the same rows among more slots, which the scan of 256 threads takes (the sums are integers)."""
import numpy as np
import pytest
import torch

from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [2304, 2305, 4095, 4096])
@pytest.mark.parametrize("n_slots", [1, 97, 256])
def test_scan_sizes(rows, n_slots):
    print("case:", rows, n_slots, flush=True)
    rng = np.random.default_rng(rows + n_slots)
    vocab = 64
    x = rng.normal(0, 3, (rows, vocab)).astype(np.float32)
    target = rng.integers(-1, vocab, rows).astype(np.int32)                  # some rows are not scored
    slot = rng.integers(0, n_slots, rows).astype(np.int32)
    x[5] = np.inf                                                            # a row whose score is not finite
    target[5] = 0
    ctx = B.Context(0)
    X, t, sl = dev(x), dev(target), dev(slot)
    score, among = torch.zeros(n_slots, device="cuda"), torch.zeros(257, device="cuda")
    ctx.sp_path_saliency(X, t, sl, n_slots, score)
    ctx.sp_path_saliency(X, t, sl, 257, among)
    torch.cuda.synchronize()
    got = score.cpu().numpy()
    assert np.array_equal(got, among.cpu().numpy()[:n_slots], equal_nan=True)
    sick = slot[5]
    assert np.isnan(got[sick])
    keep = np.arange(rows) != 5
    ref = orc.path_saliency(x[keep], target[keep], slot[keep], n_slots)
    well = np.arange(n_slots) != sick
    # rounding of the score to 32 bits, and of the fp32 logsumexp of each of its rows (magnitude below 32)
    per_slot = np.bincount(slot, minlength=n_slots)[well]
    assert np.all(np.abs(got[well] - ref[well]) <= np.abs(ref[well]) * 2.0 ** -23 + per_slot * 8 * 32 * 2.0 ** -24)
    ctx.close()
