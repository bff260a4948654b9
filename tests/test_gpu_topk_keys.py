"""Top-k order at the values and counts where its integer keys and its unrolled loop can go wrong."""
import numpy as np
import pytest
import torch

from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cap", [(1, 1), (7, 7), (8, 8), (9, 16), (63, 64), (65, 65), (257, 257), (4096, 4096), (300, 20)])
def test_order_of_special_values_and_ties(n, cap):
    print("case:", n, cap, flush=True)
    special = np.array([np.nan, np.inf, -np.inf, 0.0, -0.0, 1e-45, -1e-45, 3.4e38, -3.4e38, -np.nan, 1.0, 1.0], np.float32)
    rng = np.random.default_rng(n)
    score = np.concatenate([rng.choice(special, n), rng.normal(0, 1, 5).astype(np.float32), -np.abs(rng.choice(special, n))])
    off = np.array([0, n, n + 5, 2 * n + 5], np.int32)
    k = min(n + 3, 40)
    kept = torch.full((3, k), -7, dtype=torch.int32, device="cuda")
    ctx = B.Context(0)
    ctx.sp_prune_topk(dev(score), dev(off), 3, max(cap, 5), k, kept)
    torch.cuda.synchronize()
    for b in range(3):
        m = min(k, off[b + 1] - off[b])                    # behind the last path: -1
        ref = orc.prune_topk(score[off[b]:off[b + 1]], [0, off[b + 1] - off[b]], m)[0]
        assert np.array_equal(kept[b].cpu().numpy(), np.concatenate([ref, np.full(k - m, -1)]))
    ctx.close()
