"""The limit on the ranges of a joined cache holds for every k, also where k times the ranges of a path passes 2^31: the key
table of a workgroup has room for 120 ranges and is filled without further checks."""
import math

import numpy as np
import pytest
import torch

from paper_2404_06910_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k,status", [(100, 1, 0), (119, 1, 0), (120, 1, -3), (100, 2, -3), (100, 21474837, -3), (64, 1 << 26, -3),
                                        (1, 1 << 20, -3)])
def test_joined_range_limit(n, k, status):
    """One path of n segments that lie apart, kept k times (entries that keep nothing: -1)."""
    print("case:", n, k, flush=True)
    i32 = lambda a: np.asarray(a, np.int32)
    start = np.concatenate([[0], 5 + 2 * np.arange(n)])
    T, d = int(start[-1]) + 1, 64
    ctx = B.Context(0)
    plan = B.Plan(ctx, i32([0, n + 1]), i32(start), i32([3] + [1] * n), i32(range(-1, n)), i32([-1] + [0] * n), T, 2, 2, d, B.SP_BF16)
    z = lambda *s: torch.zeros(s, dtype=torch.bfloat16, device="cuda")
    kept = torch.full((1, k), -1, dtype=torch.int32, device="cuda")
    K, Kr, q, o = z(T, 2, d), z(1, 2, 2, d), z(1, 2, d), z(1, 2, d)
    call = lambda: ctx.sp_pruned_decode(plan, kept, k, K, K.clone(), Kr, Kr.clone(), 2, q, q.clone(), q.clone(), o, 1 / math.sqrt(d))
    if status == 0:
        call()
        torch.cuda.synchronize()
    else:
        with pytest.raises(B.SpError) as e:
            call()
        assert e.value.status == status and "disjoint ranges" in str(e.value)
    plan.close()
    ctx.close()
