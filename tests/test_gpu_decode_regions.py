"""Scratch of the decode launches that cut their key lists into pieces: every stream and every capture of a plan gets a region
of its own, however many there are and have been, and gives it back with the plan.  A captured launch tells by its grid
whether it got one: a workgroup per piece, in y."""
import threading

import numpy as np
import pytest
import torch

import sp_synth
from paper_2404_06910_amd import binding as B

from hip_graphs import Graph
from test_gpu_decode_pieces import _decode, _setup

pytestmark = pytest.mark.gpu


def _table():
    return sp_synth.forkjoin_segtable(96, [[160, 200, 180]], 24)


def _plan(ctx, seed, Hq=8, Hkv=2):
    x = _setup(ctx, np.random.default_rng(seed), "bf16", Hq, Hkv, 128, _table(), 2, [30], False, cap=40)
    o = torch.full(x["dev"]["q"].shape, float("nan"), dtype=torch.bfloat16, device="cuda")
    return x, o


def _captured(ctx, x, o, stream):
    def work():
        ctx.sp_set_stream(stream.cuda_stream)
        _decode(ctx, x, "bf16", o)
    g = Graph(stream, work)
    ctx.sp_set_stream(torch.cuda.current_stream().cuda_stream)
    return g


def test_every_capture_of_a_plan_gets_a_region():
    """70 captures on two streams, nothing eager in between (as a program that captures one graph per layer does)."""
    ctx = B.Context(0)
    x, o = _plan(ctx, 1)
    want = _decode(ctx, x, "bf16").clone()
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    graphs = [_captured(ctx, x, o, streams[i % 2]) for i in range(70)]
    assert [g.grids()[0][1] for g in graphs] == [graphs[0].grids()[0][1]] * 70
    assert all(len(g.grids()) == 1 for g in graphs) and graphs[0].grids()[0][1] > 1
    for i in (0, 3, 4, 5, 17, 69, 0):
        print("replay", i, flush=True)
        o.fill_(float("nan"))
        torch.cuda.synchronize()
        graphs[i].replay()
        torch.cuda.synchronize()
        assert torch.equal(o, want)
    for g in graphs:
        g.destroy()
    x["plan"].close()
    ctx.close()


def test_the_last_region_and_going_without():
    """256 regions to a plan, one of them the eager stream's: later captures go without, which changes no bit."""
    ctx = B.Context(0)
    x, o = _plan(ctx, 2)
    want = _decode(ctx, x, "bf16").clone()
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    graphs = [_captured(ctx, x, o, stream) for _ in range(260)]
    ys = [g.grids()[0][1] for g in graphs]
    assert ys[0] > 1 and ys == [ys[0]] * 255 + [1] * 5
    for i in (254, 255, 259):
        print("replay", i, flush=True)
        o.fill_(float("nan"))
        torch.cuda.synchronize()
        graphs[i].replay()
        torch.cuda.synchronize()
        assert torch.equal(o, want)
    for g in graphs:
        g.destroy()
    x["plan"].close()
    ctx.close()


def test_the_per_thread_stream_of_every_thread():
    """hipStreamPerThread names another stream in each host thread: launches of several threads, one after the other."""
    ctx = B.Context(0)
    x, o = _plan(ctx, 3)
    want = _decode(ctx, x, "bf16").clone()
    torch.cuda.synchronize()
    ctx.sp_set_stream(2)                                     # hipStreamPerThread
    outs = [torch.full_like(o, float("nan")) for _ in range(6)]

    def work(out):
        for _ in range(4):
            _decode(ctx, x, "bf16", out)
    torch.cuda.synchronize()
    for out in outs:
        t = threading.Thread(target=work, args=(out,))
        t.start()
        t.join()
    torch.cuda.synchronize()
    assert all(torch.equal(out, want) for out in outs)
    x["plan"].close()
    ctx.close()


def test_regions_come_back_with_the_plan():
    """A plan per request, each captured on several streams, replayed and destroyed; the graphs of a plan run on both streams
    at once, with other graphs of the same plan."""
    ctx = B.Context(0)
    streams = [torch.cuda.Stream() for _ in range(6)]
    for request in range(12):
        print("request", request, flush=True)
        x, o = _plan(ctx, request)
        want = _decode(ctx, x, "bf16").clone()
        outs = [torch.full_like(o, float("nan")) for _ in streams]
        graphs = [_captured(ctx, x, out, s) for out, s in zip(outs, streams)]
        assert all(g.grids()[0][1] > 1 for g in graphs)
        torch.cuda.synchronize()
        for _ in range(3):
            for g in graphs:
                g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(out, want) for out in outs)
        for g in graphs:
            g.destroy()
        x["plan"].close()
    ctx.close()


def test_regions_after_an_update():
    """An updated plan serves new captures and eager launches; a table with more prompts needs larger regions."""
    ctx = B.Context(0)
    x, o = _plan(ctx, 5)
    stream = torch.cuda.Stream()
    st = _table()
    for round_ in range(40):
        if round_ % 8 == 0:
            print("round", round_, flush=True)
        st2 = st if round_ % 4 else sp_synth.forkjoin_segtable(96, [[160, 200, 180]] * 3, 24)
        x["plan"].update(st2.prompt_seg_off, st2.seg_tok_start, st2.seg_tok_len, st2.seg_parent, st2.seg_path, st2.n_tokens)
        if st2 is not st:
            y = _setup(ctx, np.random.default_rng(round_), "bf16", 8, 2, 128, st2, 2, [30, 0, 9], False, cap=40)
            want = _decode(ctx, y, "bf16").clone()
            y["plan"].close()
            y["plan"] = x["plan"]
            assert torch.equal(_decode(ctx, y, "bf16"), want)
            continue
        want = _decode(ctx, x, "bf16").clone()
        g = _captured(ctx, x, o, stream)
        assert g.grids()[0][1] > 1
        o.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, want)
        g.destroy()
    x["plan"].close()
    ctx.close()


def test_a_context_without_decodes_holds_no_scratch_for_them():
    """sp_create allocates the saliency workspace alone (1.3 MB); a plan brings the regions that its own sizes need."""
    torch.cuda.synchronize()
    B.Context(0).close()                                     # whatever the runtime itself allocates once
    before = torch.cuda.mem_get_info()[0]
    ctx = B.Context(0)
    assert before - torch.cuda.mem_get_info()[0] <= 4 << 20
    ctx.close()
