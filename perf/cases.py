"""The work that a serving program has this library do, as cases that can be timed and compared.

A program of superposition prompting builds one plan per segment table, then per transformer layer calls the
ForkJoin prefill, once per request the saliency and the pruning, and per generated token and layer the decode
over the pruned cache.  A case is one such pass through the public entry points of `paper_2404_06910_amd`.

Kinds of case:
  request   the whole online pass of a request: prefill, saliency, pruning and a short response
            (five tokens, the paper's timing protocol), with the kept table staying on the device
  prefill   one layer's attention over a batch of prompts; "full" computes every row, "online" computes the
            query copies against cached documents (path caching), "round" is a later round of iterative
            superposition: the remaining documents and their query copies behind a chain of kept documents
  prune     saliency of every query row, then the top-k of the scores
  decode    one or more generated tokens for every prompt over [preamble; kept paths; response]

Shapes are those of `sp_synth.WORKLOADS` and of the tests, and sizes around them.  Everything that is shape
(document lengths, response lengths) follows from the case alone; everything that is value (tensors, targets,
kept paths) follows from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2404_06910_amd import binding as B

_BASE = {
    "kind": "prefill", "dtype": "bf16", "prompts": 1, "hq": 32, "hkv": 32, "d": 128, "preamble": 64, "paths": 20,
    "doc_lo": 128, "doc_hi": 128, "query": 24, "packing": "interleaved", "bias": False, "rows": "full", "chain": 0,
    "kv_layout": "token", "vocab": 50432, "logit_dtype": "bf16", "logit_std": 3.0, "mean": False, "prior": False,
    "k": 2, "steps": 5, "resp_max": 0,
}


def _case(name=None, **kw):
    c = dict(_BASE)
    c.update(kw)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # The smallest call of all: the four-head fp32 configuration, start to end.  Nothing but launches and
        # host work; what a test suite or a first try of the library runs.
        _case("request_tiny_f32", kind="request", dtype="f32", hq=4, hkv=4, d=64, preamble=16, paths=4, doc_lo=32,
              doc_hi=32, query=8, vocab=512, logit_dtype="f32", logit_std=2.0, k=1, steps=4),
        # One user's question over 20 retrieved documents of uneven length at the shape of a 7B model's layer:
        # what an interactive service runs, where latency counts.
        _case("request_one_prompt", kind="request", preamble=57, doc_lo=64, doc_hi=220, query=19),
        # A batch of eight such questions with documents cut to one length (the benchmark's prefill).
        _case("prefill_mha_batch", prompts=8),
        # Heavy retrieval: 64 ragged documents, a model whose positions act as a distance penalty.
        _case("prefill_ragged_bias", prompts=4, paths=64, doc_lo=64, doc_hi=256, query=32, bias=True),
        # Grouped query heads, sixteen prompts.
        _case("prefill_gqa_batch", prompts=16, hkv=8, preamble=96, doc_lo=160, doc_hi=160),
        # Path caching: documents were processed ahead of time, only the query copies are computed; the cache
        # holds the documents first and the queries behind them.
        _case("prefill_online_cached", prompts=8, rows="online", packing="grouped", doc_lo=64, doc_hi=220),
        # A later round of iterative superposition: 16 documents behind a chain of four kept ones.
        _case("prefill_iterative_round", prompts=8, rows="round", chain=4),
        # The fp32 precision path at a model's head shape (a numerical check of one request).
        _case("prefill_f32_one_prompt", dtype="f32", doc_lo=64, doc_hi=220),
        # Saliency and pruning of the eight-prompt batch, and of one prompt from an fp32 LM head with length
        # normalisation and a document prior.
        _case("prune_mha_batch", kind="prune", prompts=8),
        _case("prune_one_prompt_f32", kind="prune", logit_dtype="f32", vocab=50257, mean=True, prior=True, k=4, query=17),
        # Generation: 64 prompts in the middle of their responses, 2 of 20 paths kept ...
        _case("decode_mha_batch", kind="decode", prompts=64, steps=1, resp_max=255),
        # ... and a few prompts of a grouped-head model with four kept paths, several tokens in a row.
        _case("decode_gqa_few", kind="decode", prompts=6, hkv=8, preamble=96, doc_lo=64, doc_hi=220, k=4, steps=4,
              resp_max=120),
    ]


# Most that a drawn case of a kind may cost (bytes and flops of `work`), so that none costs more than the largest
# listed one.
_MOST_BYTES, _MOST_FLOPS, _MOST_F32_FLOPS = 1.6e9, 2.0e11, 1.2e10


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["request", "prefill", "prefill", "prefill", "prune", "decode"])
        f32 = rng.random() < 0.2
        hq, hkv, d = rng.choice([(32, 32, 128), (32, 32, 128), (32, 8, 128), (32, 8, 128), (16, 16, 64), (32, 4, 64),
                                 (24, 24, 128), (12, 6, 128)])
        if f32 and kind == "request" and rng.random() < 0.5:
            hq, hkv, d = 4, 4, 64
        lo = log_int(24, 192)
        hi = rng.choice([lo, lo, min(256, lo + log_int(8, 160))])
        paths = log_int(4, 64)
        c = _case(kind=kind, dtype="f32" if f32 else "bf16", hq=hq, hkv=hkv, d=d, preamble=log_int(12, 128), paths=paths,
                  doc_lo=lo, doc_hi=hi, query=log_int(4, 40), packing=rng.choice(["interleaved", "grouped"]),
                  bias=rng.random() < 0.3, kv_layout=rng.choice(["token", "token", "head"]),
                  vocab=rng.choice([32000, 50257, 50432, 128256, log_int(8000, 130000)]),
                  logit_dtype=rng.choice(["bf16", "bf16", "f32"]), mean=rng.random() < 0.3, prior=rng.random() < 0.3,
                  k=min(paths, rng.choice([1, 2, 4])))
        if kind == "request":
            c.update(prompts=log_int(1, 4), steps=rng.randint(2, 6))
        elif kind == "prefill":
            c.update(prompts=log_int(1, 16), rows=rng.choice(["full", "full", "online", "round"]))
            if c["rows"] == "round":
                c.update(chain=rng.randint(1, 4), paths=max(6, paths))
        elif kind == "prune":
            c.update(prompts=log_int(1, 16))
        else:
            c.update(prompts=log_int(1, 64), steps=rng.choice([1, 2, 4]), resp_max=log_int(8, 255))
        w = work(c)
        if (w["bytes"] <= _MOST_BYTES and w["flops"] <= (_MOST_F32_FLOPS if f32 else _MOST_FLOPS)
                and _state_bytes(c) <= 16e9):
            return c


# ---- shapes ------------------------------------------------------------------------------------------------------

class _Table:
    """Segment table of a case: preamble -> [chain of kept documents ->] {document -> its query copy} per prompt."""

    def __init__(self, c):
        rng = random.Random("lengths %s" % [c[k] for k in ("prompts", "paths", "doc_lo", "doc_hi", "query", "preamble")])
        off, start, length, parent, path, cached = [0], [], [], [], [], []
        P, Lq, n, tok = c["preamble"], c["query"], c["paths"], 0
        self.pairs = self.rows = self.keys = 0
        self.path_len, self.joined = [], []          # per prompt: tokens of each path; shared tokens
        self.path_off = [0]

        def seg(at, ln, par, pth, is_cached):
            start.append(at); length.append(ln); parent.append(par); path.append(pth); cached.append(int(is_cached))
            return len(start) - 1

        for _ in range(c["prompts"]):
            docs = [rng.randint(c["doc_lo"], c["doc_hi"]) for _ in range(n)]
            pool, at = [], tok + P
            if c["packing"] == "grouped":
                for ln in docs:
                    pool.append([at, 0]); at += ln
                for e in pool:
                    e[1] = at; at += Lq
            else:
                for ln in docs:
                    pool.append([at, at + ln]); at += ln + Lq
            chain = sorted(rng.sample(range(n), c["chain"]))
            rest = [i for i in range(n) if i not in chain]
            off_line = c["rows"] != "full"
            tail = seg(tok, P, -1, -1, off_line)
            for i in chain:
                tail = seg(pool[i][0], docs[i], tail, -1, True)
            shared = P + sum(docs[i] for i in chain)
            if not off_line:
                self.pairs += P * (P + 1) // 2
                self.rows += P
            self.keys += shared
            for j, i in enumerate(rest):
                ln = docs[i]
                s = seg(pool[i][0], ln, tail, j, c["rows"] == "online")
                seg(pool[i][1], Lq, s, j, False)
                if c["rows"] != "online":
                    self.pairs += ln * shared + ln * (ln + 1) // 2
                    self.rows += ln
                self.pairs += Lq * (shared + ln) + Lq * (Lq + 1) // 2
                self.rows += Lq
                self.keys += ln + Lq
            off.append(len(start))
            self.path_len.append([docs[i] + Lq for i in rest])
            self.joined.append(shared)
            self.path_off.append(self.path_off[-1] + len(rest))
            tok = at
        i32 = lambda a: np.asarray(a, np.int32)
        self.n_tokens, self.n_slots = tok, self.path_off[-1]
        self.args = (i32(off), i32(start), i32(length), i32(parent), i32(path))
        self.cached = np.asarray(cached, np.uint8) if any(cached) else None
        self.resp_len = [rng.randint(0, c["resp_max"]) for _ in range(c["prompts"])]


def _esz(dtype):
    return 2 if dtype == "bf16" else 4


def _torch_dtype(dtype):
    return torch.bfloat16 if dtype == "bf16" else torch.float32


def _state_bytes(c):
    t = _Table(c)
    n = t.n_tokens * c["d"] * 2 * (c["hq"] + c["hkv"]) * _esz(c["dtype"])
    if c["kind"] in ("request", "prune"):
        n += t.n_slots * c["query"] * c["vocab"] * _esz(c["logit_dtype"])
    return n


# ---- what a pass cannot do without ---------------------------------------------------------------------------------

def work(case):
    c, t = case, _Table(case)
    e, nbytes, flops = _esz(c["dtype"]), 0.0, 0.0
    if c["kind"] in ("request", "prefill"):
        # Q and O of the rows that are computed, K and V of every key
        nbytes += c["d"] * e * 2 * (t.rows * c["hq"] + t.keys * c["hkv"])
        flops += 4.0 * c["d"] * c["hq"] * t.pairs
    if c["kind"] in ("request", "prune"):
        rows = t.n_slots * c["query"]
        nbytes += rows * c["vocab"] * _esz(c["logit_dtype"]) + 8 * rows + 4 * t.n_slots
        flops += 4.0 * rows * c["vocab"]
    if c["kind"] in ("request", "decode"):
        keys = 0.0                                     # the kept paths are values: their mean length stands for them
        for b in range(c["prompts"]):
            mean = sum(t.path_len[b]) / len(t.path_len[b])
            for s in range(c["steps"]):
                keys += t.joined[b] + c["k"] * mean + t.resp_len[b] + s + 1
        rows = c["prompts"] * c["steps"]
        nbytes += c["d"] * e * (2 * c["hkv"] * keys + rows * (2 * c["hq"] + 4 * c["hkv"]))
        flops += 4.0 * c["d"] * c["hq"] * keys
    return {"bytes": int(nbytes), "flops": int(flops)}


def tolerance(case):
    # About four times what the path shows against the same sums in 64 bits (listed and drawn cases, largest):
    #   bf16 attention, whose probabilities and outputs are rounded to 8 bits   2.3e-3 of the norm, 2.2e-2 of the rms
    #   fp32 attention                                                          1.9e-7 of the norm, 2.5e-6 of the rms
    #   scores, sums of fp32 log-likelihoods over the vocabulary                5e-8 of the norm, 9e-8 of the rms;
    #   there an fp32 logsumexp in another order moves each term by up to a rounding of its maximum (about 1e-6)
    if case["kind"] == "prune":
        return {"rel": 1e-6, "max": 4e-6}
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 8e-2}
    return {"rel": 1e-6, "max": 1e-5}


# ---- a user's program ----------------------------------------------------------------------------------------------

_ctx = None


def _context():
    """The program's one library context, on torch's current stream."""
    global _ctx
    if _ctx is None:
        _ctx = B.Context(torch.cuda.current_device())
    return _ctx


class _State:
    pass


def prepare(case, seed):
    c, t = case, _Table(case)
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rng = np.random.default_rng(seed)
    dt, Bn, d = _torch_dtype(c["dtype"]), c["prompts"], c["d"]

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=dt)

    def cache(n):
        # token-major [n, heads, d], or a per-head cache seen as such a tensor
        if c["kv_layout"] == "head":
            return normal(c["hkv"], n, d).transpose(0, 1)
        return normal(n, c["hkv"], d)

    s = _State()
    s.case, s.ctx, s.scale, s.n_slots = c, _context(), 1.0 / math.sqrt(d), t.n_slots
    s.n_paths_max = max(len(p) for p in t.path_len)
    pos = slopes = None
    if c["bias"] and c["kind"] != "prune":
        pos = B.equilibrium_positions(*t.args, t.n_tokens)
        slopes = np.exp2(-np.linspace(1.0, 8.0, c["hq"])).astype(np.float32)
    if c["kind"] != "prune":
        s.plan = B.Plan(s.ctx, *t.args, t.n_tokens, c["hq"], c["hkv"], d, B.SP_BF16 if c["dtype"] == "bf16" else B.SP_F32,
                        tok_pos=pos, alibi_slopes=slopes, seg_cached=t.cached)
        s.K, s.V = cache(t.n_tokens), cache(t.n_tokens)
    if c["kind"] in ("request", "prefill"):
        s.Q = normal(t.n_tokens, c["hq"], d)
        s.O = torch.zeros_like(s.Q)
    if c["kind"] in ("request", "prune"):
        rows = t.n_slots * c["query"]
        per = 16 // _esz(c["logit_dtype"])             # rows start at 16-byte boundaries, as an LM head pads them
        pitch = (c["vocab"] + per - 1) // per * per
        full = torch.randn((rows, pitch), generator=g, device="cuda", dtype=_torch_dtype(c["logit_dtype"]))
        s.logits = full.mul_(c["logit_std"])[:, :c["vocab"]]
        # every path of a prompt carries a copy of the same query
        target = np.concatenate([np.tile(rng.integers(0, c["vocab"], c["query"]), len(p)) for p in t.path_len])
        s.target = torch.from_numpy(target.astype(np.int32)).cuda()
        s.row_path = torch.from_numpy(np.repeat(np.arange(t.n_slots, dtype=np.int32), c["query"])).cuda()
        s.prior = torch.from_numpy(rng.normal(-3.0, 1.0, t.n_slots).astype(np.float32)).cuda() if c["prior"] else None
        s.path_off = torch.from_numpy(np.asarray(t.path_off, np.int32)).cuda()
        s.score = torch.zeros(t.n_slots, device="cuda")
        s.kept = torch.zeros((Bn, c["k"]), dtype=torch.int32, device="cuda")
    if c["kind"] in ("request", "decode"):
        s.cap = max(t.resp_len) + c["steps"]
        s.Kr, s.Vr = normal(Bn, s.cap, c["hkv"], d), normal(Bn, s.cap, c["hkv"], d)
        s.resp_len = torch.tensor(t.resp_len, dtype=torch.int32, device="cuda")
        s.q, s.k, s.v = (normal(c["steps"], Bn, h, d) for h in (c["hq"], c["hkv"], c["hkv"]))
        s.o = torch.zeros_like(s.q)
        s.pos_resp, s.new_pos = None, [None] * c["steps"]
        if pos is not None:
            first = float(pos.max()) + 1.0
            s.pos_resp = first + torch.arange(s.cap, device="cuda", dtype=torch.float32).repeat(Bn, 1)
            s.new_pos = [first + i + s.resp_len.float() for i in range(c["steps"])]
    if c["kind"] == "decode":
        kept = np.stack([rng.permutation(len(p))[:c["k"]] for p in t.path_len])
        s.kept = torch.from_numpy(kept.astype(np.int32)).cuda()
    return s


def run(s):
    c, ctx, out = s.case, s.ctx, {}
    if c["kind"] in ("request", "prefill"):
        ctx.sp_forkjoin_prefill(s.plan, s.Q, s.K, s.V, s.O, s.scale)
        out["O"] = s.O
    if c["kind"] in ("request", "prune"):
        ctx.sp_path_saliency(s.logits, s.target, s.row_path, s.n_slots, s.score, prior=s.prior,
                             mode=B.SALIENCY_MEAN if c["mean"] else B.SALIENCY_SUM)
        ctx.sp_prune_topk(s.score, s.path_off, c["prompts"], s.n_paths_max, c["k"], s.kept)
        out["score"], out["kept"] = s.score, s.kept
    if c["kind"] in ("request", "decode"):
        for i in range(c["steps"]):
            ctx.sp_pruned_decode(s.plan, s.kept, c["k"], s.K, s.V, s.Kr, s.Vr, s.cap, s.q[i], s.k[i], s.v[i], s.o[i],
                                 s.scale, resp_len=s.resp_len, resp_len_add=i, pos_resp=s.pos_resp,
                                 new_pos=s.new_pos[i])
        out["o"], out["K_resp"], out["V_resp"] = s.o, s.Kr, s.Vr
    return out
