"""Saliency of few rows (each row cut into pieces over several workgroups) and the two ways the rows of a path are added
up, at the sizes where they change over."""
import numpy as np
import pytest
import torch

from oracle import sp_oracle as orc
from paper_2404_06910_amd import binding as B

from gpu_util import dev
import sp_synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = B.Context(0)
    yield c
    c.close()


def _scores(ctx, x, dtype, target, row_path, n_slots, **kw):
    rows, vocab = x.shape
    per = 4 if dtype == "f32" else 8
    full = torch.full((rows, (vocab + per - 1) // per * per), 50.0).numpy()   # what lies behind a row's end is not read
    full[:, :vocab] = x
    out = torch.full((n_slots,), float("nan"), device="cuda")
    ctx.sp_path_saliency(dev(full, dtype)[:, :vocab], dev(target), dev(row_path), n_slots, out, **kw)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,vecs,tail", [(1, 1023, 0), (1, 1024, 1), (3, 2047, 0), (2, 2049, 3), (5, 5000, 2),
                                            (680, 3075, 1), (1024, 2048, 0), (1025, 2050, 1)])
def test_pieces_match_the_oracle(ctx, dtype, rows, vecs, tail):
    print("case:", dtype, rows, vecs, tail, flush=True)
    vocab = vecs * (4 if dtype == "f32" else 8) + tail
    rng = np.random.default_rng(rows + vecs)
    x = sp_synth.round_to_dtype(rng.normal(0, 3, (rows, vocab)).astype(np.float32), dtype)
    target = rng.integers(0, vocab, rows).astype(np.int32)
    target[0] = vocab - 1
    if rows > 2:
        target[rows // 2] = -1
    n_slots = max(1, rows // 20)
    row_path = (np.arange(rows) * n_slots // rows).astype(np.int32)
    got = _scores(ctx, x, dtype, target, row_path, n_slots)
    ref = orc.path_saliency(x, target, row_path, n_slots)
    # a row's lp is a few fp32 roundings of a logsumexp below 32 in magnitude, and a slot has at most 41 rows
    assert np.abs(got - ref).max() <= 41 * 4 * 32 * 2.0 ** -24
    assert np.array_equal(got, _scores(ctx, x, dtype, target, row_path, n_slots))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_values_that_are_not_finite_in_any_piece(ctx, dtype):
    rng = np.random.default_rng(8)
    vocab = 8 * 1024 * 4 + 5
    x = sp_synth.round_to_dtype(rng.normal(0, 2, (7, vocab)).astype(np.float32), dtype)
    target = np.full(7, 77, np.int32)
    x[1, vocab - 1] = np.nan                   # scalar tail
    x[2, 20000] = np.inf                       # a middle piece
    x[3, 77] = -np.inf                         # the target itself
    x[4, :] = -np.inf                          # nothing at all
    x[5, 4096:] = -np.inf                      # whole pieces of the row
    x[6, :] = -np.inf; x[6, 30000] = 1.5; target[6] = 30000
    got = _scores(ctx, x, dtype, target, np.arange(7, dtype=np.int32), 7)
    ref = orc.path_saliency(x[[0, 5]], target[[0, 5]], np.arange(2, dtype=np.int32), 2)
    assert np.abs(got[[0, 5]] - ref).max() <= 4 * 32 * 2.0 ** -24
    assert np.isnan(got[1]) and np.isnan(got[2]) and got[3] == -np.inf and np.isnan(got[4])
    assert got[6] == 0.0


@pytest.mark.parametrize("rows,n_slots", [(4096, 300), (7168, 512)])
def test_scan_and_atomic_sums_agree_bit_for_bit(ctx, rows, n_slots):
    """The most rows that the scan takes (more where there are many slots); one more row, without a target, goes through
    the atomics."""
    rng = np.random.default_rng(9)
    vocab = 40
    x = rng.normal(0, 3, (rows + 1, vocab)).astype(np.float32)
    target = rng.integers(0, vocab, rows + 1).astype(np.int32)
    target[rng.integers(0, rows, 500)] = -1
    target[rows] = -1
    row_path = rng.integers(-2, n_slots + 2, rows + 1).astype(np.int32)      # out of range: the nearest slot
    prior = dev(rng.normal(size=n_slots).astype(np.float32))
    for mode in (B.SALIENCY_SUM, B.SALIENCY_MEAN):
        a = _scores(ctx, x[:rows], "f32", target[:rows], row_path[:rows], n_slots, mode=mode, prior=prior)
        b = _scores(ctx, x, "f32", target, row_path, n_slots, mode=mode, prior=prior)
        assert np.array_equal(a, b)
    big = 4096                                  # slots: the same rows, but more path numbers than the scan reads
    a = _scores(ctx, x[:1024], "f32", target[:1024], row_path[:1024], big)
    b = _scores(ctx, x[:1025], "f32", np.where(np.arange(1025) < 1024, target[:1025], -1).astype(np.int32),
                row_path[:1025], big)
    assert np.array_equal(a, b)
