"""The work a serving program has the prefix store do, as measurable cases.

Four kinds of call, each through the binding's public entry points:

  load    requests (a popular passage, then text of their own) are looked up
          and the matched blocks' KV is copied into the caller's paged cache,
          in one fused call or layer by layer from one prepared list
  query   the longest-prefix query alone, ragged requests against stored
          documents: what a scheduler asks before it places a request
  walk    requests that branch everywhere (agents, trees of thought): walks
          down a prefix tree, looked up alone or loaded too
  insert  a full, evicting store takes the blocks a batch of requests adds
          and their KV is scattered from the paged cache into the pool

The KV shapes are those of the repository's own configurations. Every output
is whole numbers or copied bytes, so all comparisons are exact. Block tables
are random permutations: the free list of a paged cache that has been in use.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_22648_amd.ptstore import PTSTORE_FLAG_EVICT, PrefixStore, StoreShape

VOCAB = 32000
#: layers, KV heads, head size (2-byte elements)
SHAPES = {
    "tiny": (2, 8, 128),
    "8b": (32, 8, 128),
    "70b": (80, 8, 128),
    "hybrid": (32, 8, 128),   # layers alternate 8 and 2 KV heads
    "onelayer": (1, 8, 128),
    "index": (1, 1, 16),      # next to no payload: the index is what is asked
}


def listed():
    return [
        # one user's short prompt on a small model: the smallest call, all latency
        dict(name="load_one_tiny", kind="load", shape="tiny", requests=1, stored=16, population=16,
             passage=768, suffix=256, zipf=1.0, page=16, ragged=False, layerwise=False, host=0.0),
        # a batch of short prompts on a small model, half of the passages popular enough to be stored
        dict(name="load_batch_tiny", kind="load", shape="tiny", requests=64, stored=16, population=32,
             passage=768, suffix=256, zipf=1.0, page=16, ragged=False, layerwise=False, host=0.0),
        # one request at a time on an 8B-shaped model, of odd length
        dict(name="load_one_8b", kind="load", shape="8b", requests=1, stored=16, population=16,
             passage=2805, suffix=128, zipf=1.0, page=16, ragged=False, layerwise=False, host=0.0),
        # a prefill batch of long-passage questions on an 8B-shaped model
        dict(name="load_batch_8b", kind="load", shape="8b", requests=48, stored=64, population=128,
             passage=3584, suffix=512, zipf=1.1, page=16, ragged=False, layerwise=False, host=0.0),
        # the same model loading layer by layer, so that each layer's compute can follow its copy
        dict(name="load_layers_8b", kind="load", shape="8b", requests=16, stored=32, population=48,
             passage=3584, suffix=512, zipf=1.1, page=16, ragged=False, layerwise=True, host=0.0),
        # a hybrid model, whose layers' slabs differ in size
        dict(name="load_hybrid", kind="load", shape="hybrid", requests=32, stored=32, population=64,
             passage=3584, suffix=512, zipf=1.1, page=16, ragged=False, layerwise=False, host=0.0),
        # long contexts on a 70B-shaped model, a part of the store in pinned host memory
        dict(name="load_tiered_70b", kind="load", shape="70b", requests=2, stored=4, population=4,
             passage=7680, suffix=512, zipf=0.5, page=16, ragged=False, layerwise=False, host=0.05),
        # a scheduler's query for ragged requests against ragged documents, 32-token pages
        dict(name="query_ragged", kind="query", requests=96, documents=64, longest=16384, page=32),
        # the query for many branching requests against a million stored blocks
        dict(name="query_walks", kind="walk", shape="index", requests=8192, roots=64, capacity=1000000,
             load=False),
        # branching requests loaded too: one-layer blocks, a few rows shared by very many requests
        dict(name="load_walks", kind="walk", shape="onelayer", requests=4096, roots=16, capacity=131072,
             load=True),
        # chat turns on a small model: each request adds one or two blocks to what is stored
        dict(name="insert_turns_tiny", kind="insert", shape="tiny", requests=128, stored=16, passage=3584,
             fresh_lo=1, fresh_hi=2, repeat=0.25, slack=1536, ring=24),
        # whole questions on an 8B-shaped model: each request adds 512 tokens
        dict(name="insert_questions_8b", kind="insert", shape="8b", requests=32, stored=16, passage=3584,
             fresh_lo=32, fresh_hi=32, repeat=0.0, slack=2560, ring=6),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: odd sizes, ragged requests, other page sizes."""
    kind = rng.choice(["load", "load", "load", "load", "query", "walk", "insert", "insert"])
    if kind == "load":
        shape = rng.choice(["tiny", "tiny", "8b", "8b", "70b", "hybrid"])
        page = rng.choice([16, 16, 32, 8])
        # at most about 16 GB of paged cache
        block = 2 * sum(_heads(shape)) * 128 * 2 * page
        passage = _log_int(rng, 200, 8000 if shape == "70b" else 4000)
        suffix = _log_int(rng, 16, 600)
        blocks = (passage + suffix) // page
        most = max(1, min(128, (16 << 30) // (blocks * block)))
        requests = _log_int(rng, 1, most)
        stored = max(1, min(64, (16 << 30) // max(1, (passage // page) * block)))
        stored = _log_int(rng, min(4, stored), stored)
        return dict(kind=kind, shape=shape, requests=requests, stored=stored,
                    population=stored + int(stored * rng.uniform(0, 1)), passage=passage, suffix=suffix,
                    zipf=round(rng.uniform(0.5, 1.2), 2), page=page, ragged=rng.random() < 0.5,
                    layerwise=rng.random() < 0.25, host=rng.choice([0.0, 0.0, 0.0, 0.02]))
    if kind == "query":
        return dict(kind=kind, requests=_log_int(rng, 1, 256), documents=_log_int(rng, 8, 128),
                    longest=_log_int(rng, 600, 16384), page=rng.choice([16, 32, 64, 24]))
    if kind == "walk":
        load = rng.random() < 0.5
        requests = _log_int(rng, 60, 3000 if load else 8192)
        return dict(kind=kind, shape="onelayer" if load else "index", requests=requests,
                    roots=_log_int(rng, 4, 64), capacity=_log_int(rng, 20000, 130000 if load else 1000000),
                    load=load)
    shape = rng.choice(["tiny", "tiny", "hybrid", "8b"])
    small = shape == "tiny"
    requests = _log_int(rng, 1, 128 if small else 24)
    lo = rng.choice([1, 1, 8]) if small else rng.choice([1, 16, 32])
    hi = lo + rng.choice([0, 1, 5])
    # room for three batches: the blocks of the ring's oldest batch are gone when it comes round again
    return dict(kind=kind, shape=shape, requests=requests, stored=_log_int(rng, 4, 16),
                passage=_log_int(rng, 400, 3584), fresh_lo=lo, fresh_hi=hi,
                repeat=rng.choice([0.0, 0.25]), slack=max(64, 3 * requests * hi), ring=24 if hi < 8 else 6)


# --- shapes -----------------------------------------------------------------


def _heads(shape):
    layers, heads, _ = SHAPES[shape]
    return [8, 2] * (layers // 2) if shape == "hybrid" else [heads] * layers


def _block_bytes(shape, page=16):
    return 2 * sum(_heads(shape)) * SHAPES[shape][2] * 2 * page


def _store_shape(shape, page=16):
    layers, heads, dim = SHAPES[shape]
    slabs = None
    if shape == "hybrid":
        slabs = tuple(h * page * dim * 2 for h in _heads(shape))
    return StoreShape(layers, heads, dim, page, 2, slabs)


def _zipf(n, s):
    p = np.arange(1, n + 1, dtype=np.float64) ** -s
    return p / p.sum()


# --- inputs -----------------------------------------------------------------


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _tokens(g, *size):
    return torch.randint(0, VOCAB, size, dtype=torch.int32, device="cuda", generator=g)


def _bytes(g, n):
    """n random bytes, as 8-byte words."""
    return torch.empty(n // 8, dtype=torch.int64, device="cuda").random_(generator=g)


def _table(g, requests, blocks):
    """Every request's pages, scattered over the paged cache."""
    return torch.randperm(requests * blocks, device="cuda", generator=g).to(torch.int32).view(requests, blocks)


def _pack(rows, lengths):
    """[R, longest] tokens cut to `lengths` (host array): CSR tokens and offsets."""
    n = torch.from_numpy(np.asarray(lengths, dtype=np.int64)).cuda()
    at = torch.arange(rows.shape[1], device="cuda")
    offsets = torch.zeros(len(lengths) + 1, dtype=torch.int64, device="cuda")
    torch.cumsum(n, 0, out=offsets[1:])
    return rows[at[None, :] < n[:, None]].contiguous(), offsets


def _fill(store, g):
    """Random KV in every block the store has room for (as earlier scatters left it)."""
    store.pool_tensor().view(torch.int64).random_(generator=g)
    b = store.buffers()
    if b.host_blocks:
        host = store.host_tensor()
        host.view(torch.int64).copy_(_bytes(g, host.numel()).view(host.shape[0], -1))


def _prefix_then_own(g, source, picked, keep, own, longest):
    """Rows of `longest` tokens: source[picked][:keep], then tokens of their own; and their lengths."""
    rows = _tokens(g, len(picked), longest)
    width = min(longest, source.shape[1])
    at = torch.arange(width, device="cuda")
    kept = torch.from_numpy(np.asarray(keep, dtype=np.int64)).cuda()
    src = source[torch.from_numpy(np.asarray(picked, dtype=np.int64)).cuda()][:, :width]
    rows[:, :width] = torch.where(at[None, :] < kept[:, None], src, rows[:, :width])
    return _pack(rows, np.minimum(np.asarray(keep) + np.asarray(own), longest))


def _prepare_load(c, seed):
    g, host_rng = _generator(seed), np.random.default_rng(seed)
    page, R = c["page"], c["requests"]
    per = c["passage"] // page
    passages = _tokens(g, c["population"], c["passage"])
    picked = host_rng.choice(c["population"], size=R, p=_zipf(c["population"], c["zipf"]))
    if R == 1:  # the one request is a hit
        picked[:] = host_rng.integers(0, c["stored"])
    keep, own = np.full(R, c["passage"]), np.full(R, c["suffix"])
    if c["ragged"]:
        keep = host_rng.integers(min(page, c["passage"]), c["passage"] + 1, size=R)
        own = host_rng.integers(0, c["suffix"] + 1, size=R)
    longest = c["passage"] + c["suffix"]
    tokens, offsets = _prefix_then_own(g, passages, picked, keep, own, longest)
    blocks = longest // page
    room = max(1, c["stored"] * per)
    in_host = int(room * c["host"])
    replicas = min(in_host // 4, (room - in_host) // 2)
    store = PrefixStore(_store_shape(c["shape"], page), room - in_host + replicas, host_blocks=in_host,
                        replica_blocks=replicas, flags=PTSTORE_FLAG_EVICT if in_host else 0)
    st, so = _pack(passages[:c["stored"]], np.full(c["stored"], c["passage"]))
    store.insert(st, so, max(1, per))
    _fill(store, g)
    if replicas:
        store.lookup(tokens, offsets, blocks)
        store.replicate()
    cache = torch.zeros(R * blocks * store.shape.block_bytes // 8, dtype=torch.int64, device="cuda")
    return dict(case=c, store=store, tokens=tokens, offsets=offsets, blocks=blocks,
                table=_table(g, R, blocks), cache=cache)


def _prepare_query(c, seed):
    g, host_rng = _generator(seed), np.random.default_rng(seed)
    page, D, R = c["page"], c["documents"], c["requests"]
    lengths = np.exp(host_rng.uniform(np.log(4 * page), np.log(c["longest"]), size=D)).astype(np.int64)
    documents = _tokens(g, D, c["longest"])
    blocks = max(1, c["longest"] // page)
    store = PrefixStore(_store_shape("index", page), D * blocks)
    st, so = _pack(documents, lengths)
    store.insert(st, so, blocks)
    picked = host_rng.integers(0, D, size=R)
    keep = (host_rng.uniform(0.2, 1.0, size=R) * lengths[picked]).astype(np.int64)
    own = host_rng.integers(0, 512, size=R)
    tokens, offsets = _prefix_then_own(g, documents, picked, keep, own, c["longest"])
    return dict(case=c, store=store, tokens=tokens, offsets=offsets, blocks=blocks)


def _mix(x):
    """SplitMix64's finaliser on int64 tensors."""
    x = x ^ ((x >> 30) & ((1 << 34) - 1))
    x = x * -0x40A7B892E31B1A47
    x = x ^ ((x >> 27) & ((1 << 37) - 1))
    x = x * -0x6B2FB644ECCEEE15
    return x ^ ((x >> 31) & ((1 << 33) - 1))


DEPTH, BRANCH, FANOUT = 64, 0.04, 4


def _walks(g, n, roots, seed):
    """n walks of DEPTH 16-token blocks down the tree that `seed` names: a node has FANOUT
    children with probability BRANCH, else one, and its tokens are a function of its path."""
    base = torch.arange(1, roots + 1, device="cuda", dtype=torch.int64) + (seed + 1) * 1000003
    h = _mix(base)[torch.randint(0, roots, (n,), device="cuda", generator=g)]
    at = torch.arange(1, 17, device="cuda", dtype=torch.int64) * -0x2E4AB5CD2E6D12FD
    out = torch.empty(n, DEPTH, 16, dtype=torch.int32, device="cuda")
    for level in range(DEPTH):
        out[:, level] = ((_mix(h[:, None] ^ at[None, :]) & 0x7FFFFFFF) % VOCAB).to(torch.int32)
        wide = ((_mix(h ^ 0x20761D6478BD642F) >> 40) & 0xFFFFFF) < int(BRANCH * (1 << 24))
        pick = torch.randint(0, FANOUT, (n,), device="cuda", generator=g)
        h = _mix(h * 0x100000001B3 + torch.where(wide, pick, torch.zeros_like(pick)) + 1)
    offsets = torch.arange(n + 1, device="cuda", dtype=torch.int64) * (DEPTH * 16)
    return out.view(-1), offsets


def _prepare_walk(c, seed):
    g = _generator(seed)
    store = PrefixStore(_store_shape(c["shape"]), c["capacity"])
    for _ in range(3):
        st, so = _walks(g, 16384, c["roots"], seed)
        store.insert(st, so, DEPTH)
    tokens, offsets = _walks(g, c["requests"], c["roots"], seed)
    s = dict(case=c, store=store, tokens=tokens, offsets=offsets, blocks=DEPTH)
    if c["load"]:
        _fill(store, g)
        s["table"] = _table(g, c["requests"], DEPTH)
        s["cache"] = torch.zeros(c["requests"] * DEPTH * store.shape.block_bytes // 8, dtype=torch.int64,
                                 device="cuda")
    return s


def _prepare_insert(c, seed):
    g, host_rng = _generator(seed), np.random.default_rng(seed)
    R, per = c["requests"], c["passage"] // 16
    passages = _tokens(g, c["stored"], per * 16)
    blocks = per + c["fresh_hi"]
    store = PrefixStore(_store_shape(c["shape"]), c["stored"] * per + c["slack"], flags=PTSTORE_FLAG_EVICT)
    st, so = _pack(passages, np.full(c["stored"], per * 16))
    store.insert(st, so, per)
    _fill(store, g)
    batches = []
    for _ in range(c["ring"]):  # each adds its own branches, so that none finds an earlier batch's
        picked = host_rng.choice(c["stored"], size=R, p=_zipf(c["stored"], 1.1))
        keep = 16 * host_rng.integers(1, per + 1, size=R)
        own = 16 * host_rng.integers(c["fresh_lo"], c["fresh_hi"] + 1, size=R)
        rows, _ = _prefix_then_own(g, passages, picked, keep, np.full(R, blocks * 16), blocks * 16)
        again = host_rng.random(R) < c["repeat"]  # requests that another of the batch repeats
        src = np.where(again, host_rng.integers(0, R, size=R), np.arange(R))
        rows = rows.view(R, blocks * 16)[torch.from_numpy(src).cuda()]
        batches.append(_pack(rows, (keep + own)[src]))
    for tokens, offsets in batches:  # the store as it is after a while: full, evicting
        store.insert(tokens, offsets, blocks)
    cache = _bytes(g, R * blocks * store.shape.block_bytes)
    parent, kept = store.meta_tensors()
    freq, prio = store.evict_tensors()
    held = dict(pool=store.pool_tensor().view(torch.int64), parent=parent, tokens=kept, freq=freq, prio=prio)
    for view in held.values():  # no copies: the store's memory, so it lives as long as they do
        view.store = store
    return dict(case=c, store=store, batches=batches, turn=0, blocks=blocks, table=_table(g, R, blocks),
                cache=cache, held=held)


def prepare(case, seed):
    make = {"load": _prepare_load, "query": _prepare_query, "walk": _prepare_walk, "insert": _prepare_insert}
    return make[case["kind"]](case, seed)


# --- one pass ---------------------------------------------------------------


def run(state):
    c, store = state["case"], state["store"]
    if c["kind"] == "insert":
        tokens, offsets = state["batches"][state["turn"] % len(state["batches"])]
        state["turn"] += 1
        m, ids, created = store.insert(tokens, offsets, state["blocks"])
        store.scatter(ids, created, state["table"], state["cache"])
        return dict(m=m, ids=ids, created=created, **state["held"])
    if c["kind"] == "query" or (c["kind"] == "walk" and not c["load"]):
        m, ids = store.lookup(state["tokens"], state["offsets"], state["blocks"])
        return dict(m=m, ids=ids)
    if c.get("layerwise"):
        m, ids = store.lookup(state["tokens"], state["offsets"], state["blocks"])
        store.gather_prepare(ids, m, state["table"], state["cache"])
        for layer in range(store.shape.layers):
            store.gather_prepared(state["cache"], (layer, layer + 1))
    else:
        m, ids = store.lookup_gather(state["tokens"], state["offsets"], state["blocks"], state["table"],
                                     state["cache"])
    return dict(m=m, ids=ids, cache=state["cache"])


# --- what a pass cannot do without ------------------------------------------


def work(case):
    c = case
    R, page = c["requests"], c.get("page", 16)
    if c["kind"] == "load":
        per = c["passage"] // page
        share = 0.5 if c["ragged"] else 1.0
        p = _zipf(c["population"], c["zipf"])[:c["stored"]]
        hits = R * p.sum() if R > 1 else 1.0
        distinct = (1 - (1 - p) ** R).sum() if R > 1 else 1.0
        moved = (hits + distinct) * per * share * _block_bytes(c["shape"], page)
        asked = R * ((c["passage"] + c["suffix"]) // page) * (4 * page + 4)
        return {"bytes": float(moved + asked + distinct * per * (4 * page + 16)), "flops": 0.0}
    if c["kind"] == "query":
        span = math.log(c["longest"]) - math.log(4 * page)
        mean = 0.6 * (c["longest"] - 4 * page) / max(span, 1e-9) + 256
        return {"bytes": float(R * mean * 4 * 2 + R * (c["longest"] // page) * 4), "flops": 0.0}
    if c["kind"] == "walk":
        nodes = c["roots"] * (1 + (FANOUT - 1) * BRANCH) ** np.arange(DEPTH)
        distinct = min(c["capacity"], float((nodes * (1 - (1 - 1 / nodes) ** R)).sum()))
        total = R * DEPTH * (64 + 4) + distinct * (64 + 16)
        if c["load"]:
            total += (R * DEPTH + distinct) * _block_bytes(c["shape"])
        return {"bytes": float(total), "flops": 0.0}
    per = c["passage"] // 16
    fresh = (c["fresh_lo"] + c["fresh_hi"]) / 2
    new = R * (1 - c["repeat"]) * fresh
    asked = R * ((per + 1) / 2 + fresh) * 64 + R * (per + c["fresh_hi"]) * 5
    return {"bytes": float(asked + new * (84 + 2 * _block_bytes(c["shape"]))), "flops": 0.0}


def tolerance(case):
    return "exact"
