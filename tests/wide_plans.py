"""Segment tables of the kind that the wide bf16 prefill takes: prompts whose paths fork behind a long chain of segments."""
import numpy as np


def chain_table(prompts, chain, docs, query=0, gap=0, cached_chain=False, query_apart=False, hole=0):
    """Every prompt: a chain of segments of the lengths `chain`, `gap` uncovered tokens behind each (so that they are as many
    key ranges), then a fork of one path per entry of `docs`, with `query` tokens behind each document (in a place of their
    own with `query_apart`; with `hole`, that many cached tokens between the two).  Returns ((seg_off, start, length, parent,
    path), n_tokens, cached flags or None)."""
    off, start, length, parent, path, cached, tok = [0], [], [], [], [], [], 0

    def seg(at, n, par, pth, is_cached=False):
        start.append(at); length.append(n); parent.append(par); path.append(pth); cached.append(is_cached)
        return len(start) - 1

    for _ in range(prompts):
        tail = -1
        for n in chain:
            tail = seg(tok, n, tail, -1, cached_chain)
            tok += n + gap
        apart = tok + sum(docs) if query_apart else 0
        for j, n in enumerate(docs):
            d = seg(tok, n, tail, j)
            tok += n
            if hole:
                d = seg(tok, hole, d, j, True)
                tok += hole
            if query and not query_apart:
                seg(tok, query, d, j)
                tok += query + gap
            elif query:
                seg(apart, query, d, j)
                apart += query
        if query_apart:
            tok = apart
        tok += gap
        off.append(len(start))
    i32 = lambda a: np.asarray(a, np.int32)
    return (i32(off), i32(start), i32(length), i32(parent), i32(path)), tok, \
        np.asarray(cached, np.uint8) if any(cached) else None


# (query heads, KV heads, table): one and two heads per workgroup; pieces of 1, 2 and 4 blocks; tiles of one group and of
# several; 1 to 15 ranges; rows and chains that end on a block or stage and just before or behind one; groups with rows before
# and behind a cached segment, in one tile and in two
CASES = {
    "siblings": (32, 32, dict(prompts=8, chain=[600], docs=[128] * 12, query=24)),
    "ragged": (32, 32, dict(prompts=7, chain=[577], docs=[1, 31, 32, 33, 63, 64, 65, 150, 97, 220, 256, 257], query=5, gap=3)),
    "ranges": (24, 24, dict(prompts=9, chain=[64, 128, 1, 200, 230], docs=[100, 17, 130, 8, 64, 90, 128, 40], query=24, gap=2,
                            cached_chain=True)),
    "most_ranges": (32, 32, dict(prompts=6, chain=[45] * 15, docs=[256, 250, 512, 500, 241, 230], query=0, gap=1,
                                 cached_chain=True)),
    "query_apart": (32, 32, dict(prompts=6, chain=[704], docs=[256, 250, 512], query=230, query_apart=True)),
    "two_heads": (12, 6, dict(prompts=10, chain=[1100, 300], docs=[220, 100, 33, 64, 150, 31, 129, 128], query=24, gap=2)),
    "holes": (32, 32, dict(prompts=10, chain=[1500], docs=[40] * 10, query=40, hole=100, cached_chain=True)),
    "holes_ragged": (24, 24, dict(prompts=9, chain=[1800, 700], docs=[24, 72, 40, 1, 32, 64, 100, 33, 24, 260, 72, 24], query=24,
                                  gap=1, hole=60, cached_chain=True)),
    "holes_of_pairs": (12, 6, dict(prompts=10, chain=[2000], docs=[24, 72, 40, 8, 100, 24], query=40, hole=33, cached_chain=True)),
    "five_by_two": (20, 10, dict(prompts=8, chain=[1111], docs=[220, 100, 1, 70, 200, 32], query=24)),
}
