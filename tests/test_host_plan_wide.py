"""Plans that the wide bf16 prefill takes: that the rule takes them, and that their work covers every row and head once."""
import numpy as np
import pytest

import bench
import sp_synth
from paper_2404_06910_amd import binding as B

from test_host_plan import _check_work_list
from wide_plans import CASES, chain_table

WIDE_SLOTS = 256                              # one workgroup per compute unit (the other kernel: 1024 or 512)


def _slots(args, T, Hq, Hkv, d=128, dtype=B.SP_BF16, cached=None):
    p = B.Plan(None, *args, T, Hq, Hkv, d, dtype, seg_cached=cached)
    n = len(p.work_items()[1]) - 1
    p.close()
    return n


@pytest.mark.parametrize("name", sorted(CASES))
def test_wide_work_list_covers_every_row_and_head_once(name):
    Hq, Hkv, kw = CASES[name]
    args, T, cached = chain_table(**kw)
    assert _slots(args, T, Hq, Hkv, cached=cached) == WIDE_SLOTS
    names = ("prompt_seg_off", "seg_tok_start", "seg_tok_len", "seg_parent", "seg_path")
    _check_work_list(dict(zip(names, args), n_tokens=T), Hq, Hkv, cached=cached)


def test_plans_that_stay_with_the_other_kernel():
    args, T, _ = chain_table(prompts=8, chain=[600], docs=[128] * 12, query=24)
    assert _slots(args, T, 32, 32, d=64) != WIDE_SLOTS
    assert _slots(args, T, 32, 8) != WIDE_SLOTS                     # four heads per workgroup
    args, T, _ = chain_table(prompts=1, chain=[600], docs=[128] * 12, query=24)
    assert _slots(args, T, 32, 32) != WIDE_SLOTS                    # too little work
    args, T, cached = chain_table(prompts=12, chain=[45] * 16, docs=[130] * 8, gap=1, cached_chain=True)
    assert _slots(args, T, 32, 32, cached=cached) != WIDE_SLOTS     # more ranges than a tile has
    wl = sp_synth.WORKLOADS["c2_mha7b_bf16"]
    st = sp_synth.forkjoin_segtable(wl.preamble_len, [[wl.doc_len] * wl.n_paths] * wl.n_prompts, wl.query_len)
    assert _slots((st.prompt_seg_off, st.seg_tok_start, st.seg_tok_len, st.seg_parent, st.seg_path), st.n_tokens, 32, 32) != WIDE_SLOTS
    # query copies behind cached documents: a wave would compute on few of its tile's stages
    args, T, _ = chain_table(prompts=8, chain=[64], docs=[128] * 20, query=24)
    cached = np.ones(len(args[1]), np.uint8)
    cached[np.flatnonzero(args[2] == 24)] = 0
    assert _slots(args, T, 32, 32, cached=cached) != WIDE_SLOTS


# Few tiles per compute unit, us with the other kernel and with the wide one
@pytest.mark.parametrize("Hq,Hkv,prompts,chain,docs,query,wide", [
    (32, 32, 3, 4096, [128] * 3, 24, False),                        # 152 / 217: an eighth of the units has two tiles
    (32, 16, 7, 2241, [25] * 3, 40, False),                         # 94 / 138: three in ten, most of them half empty
    (32, 32, 5, 8192, [40] * 6, 8, False),                          # 350 / 443: a quarter
    (32, 32, 6, 2524, [10] * 5, 40, False),                         # 112 / 152: half, and half tiles
    (24, 24, 7, 3329, [705], 24, False),                            # 321 / 369: a quarter has four, the others three
    (32, 32, 1, 32768, [250] * 4, 0, True),                         # 1060 / 933: half of the units has one, the others none
    (32, 32, 1, 16384, [250] * 8, 0, True),                         # 646 / 548: one each
])
def test_few_tiles_go_where_the_slowest_unit_ends_first(Hq, Hkv, prompts, chain, docs, query, wide):
    args, T, cached = chain_table(prompts=prompts, chain=[chain], docs=docs, query=query, gap=1, cached_chain=True)
    assert (_slots(args, T, Hq, Hkv, cached=cached) == WIDE_SLOTS) == wide
    names = ("prompt_seg_off", "seg_tok_start", "seg_tok_len", "seg_parent", "seg_path")
    if T < 60000 and not wide:
        _check_work_list(dict(zip(names, args), n_tokens=T), Hq, Hkv, cached=cached)


def test_the_benchmark_names_the_kernel_that_the_plan_takes():
    for prompts, name in ((8, "prefill_wide_kernel"), (1, "prefill_bf16_kernel")):
        args, T, _ = chain_table(prompts=prompts, chain=[600], docs=[128] * 12, query=24)
        for heads in ((32, 32), (32, 8)):                           # grouped heads: two slots per compute unit
            p = B.Plan(None, *args, T, *heads, 128, B.SP_BF16)
            assert bench._prefill_kernel(p, 256) == (name if heads == (32, 32) else "prefill_bf16_kernel")
            p.close()
