"""Saliency with (almost) no rows and very many path slots: every slot still gets its score, whichever of the two summing
kernels the sizes select, and no size is refused by a launch limit."""
import numpy as np
import pytest
import torch

from paper_2404_06910_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu

READS = 1 << 22          # row-slot pairs up to which one workgroup per slot scans the rows


@pytest.mark.parametrize("rows,n_slots", [(0, 1), (0, 16385), (0, READS), (0, READS + 1), (0, 1 << 24), (1, READS),
                                          (1, READS + 1), (3, READS // 3), (3, READS // 3 + 1), (100, 16384)])
def test_every_slot_gets_its_score(rows, n_slots):
    print("case:", rows, n_slots, flush=True)
    ctx = B.Context(0)
    rng = np.random.default_rng(rows)
    vocab = 16
    x = rng.normal(0, 2, (max(rows, 1), vocab)).astype(np.float32)
    target = rng.integers(0, vocab, max(rows, 1)).astype(np.int32)
    slot = np.linspace(0, n_slots - 1, max(rows, 1)).astype(np.int32)        # the last row: the last slot
    prior = torch.arange(n_slots, device="cuda", dtype=torch.float32)
    X, tg, sl = dev(x)[:rows], dev(target)[:rows], dev(slot)[:rows]
    score = torch.full((n_slots,), float("nan"), device="cuda")
    if rows == 0:                                            # a pointer is still required
        X = dev(x)
        st = B.lib().sp_path_saliency(ctx._h, X.data_ptr(), B.SP_F32, 0, vocab, vocab, dev(target).data_ptr(),
                                      dev(slot).data_ptr(), prior.data_ptr(), n_slots, 0, score.data_ptr())
        assert st == 0, B.lib().sp_last_error(ctx._h)
    else:
        ctx.sp_path_saliency(X, tg, sl, n_slots, score, prior=prior)
    torch.cuda.synchronize()
    got = score.cpu().numpy().astype(np.float64)
    want = np.arange(n_slots, dtype=np.float64)
    xs = x.astype(np.float64)
    lp = xs[np.arange(max(rows, 1)), target] - np.log(np.exp(xs).sum(1))
    np.add.at(want, slot[:rows], lp[:rows])
    # one fp32 rounding of slot number plus score, and the few of a logsumexp below 8 in magnitude
    assert np.abs(got - want).max() <= n_slots * 2.0 ** -24 + 8 * 8 * 2.0 ** -24
    ctx.close()
