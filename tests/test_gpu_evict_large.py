"""Evicting inserts into stores above the size that one workgroup evicts, and what a small batch
pays in them. Results against the CPU oracle, bit-exact."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_22648_amd import ptstore as P
    from tests.twin import DEV, Twin

    EVICT = P.PTSTORE_FLAG_EVICT

BT = 4


def _full_store(capacity):
    """A full evicting store of `capacity` blocks on random tokens, 64 to a request, and the rest of
    the generator's stream."""
    g = torch.Generator(device=DEV)
    g.manual_seed(11)
    s = P.PrefixStore(P.StoreShape(1, 1, 8, BT), capacity, flags=EVICT)
    left = capacity
    while left:
        n = min(left, 1 << 18)
        _insert(s, g, n // 64 or 1, min(n, 64))
        left -= (n // 64 or 1) * min(n, 64)
    s.set_timing(True)
    return s, g


def _insert(s, g, R, blocks):
    """Inserts R requests of new tokens; the insert's time in us."""
    toks = torch.randint(0, 1 << 30, (R * blocks * BT,), dtype=torch.int32, device=DEV, generator=g)
    offs = torch.arange(R + 1, dtype=torch.int64, device=DEV) * (blocks * BT)
    torch.cuda.synchronize()
    s.insert(toks, offs, blocks)
    return s.kernel_times(P.KIND_INSERT)[0] * 1e3


@pytest.mark.parametrize("capacity", [5000, 17000])
def test_one_request_inserts_rebuild_the_index(capacity):
    """One request at a time until deleted slots have made two rebuilds: each insert's results, and
    after a rebuild every block is found again."""
    rng = np.random.default_rng(capacity)
    t = Twin(1, 1, 8, BT, capacity, flags=EVICT, payload=False)
    kept = []
    for i in range(6 * capacity // 64):
        seq = rng.integers(0, 1 << 30, size=64 * BT, dtype=np.int32)
        offs = np.array([0, seq.size], dtype=np.int64)
        before = t.gpu.stats()["index_rebuilds"]
        t.insert(seq, offs, 64)
        kept.append(seq)
        if t.gpu.stats()["index_rebuilds"] > before:
            recent = kept[-capacity // 64 - 8:]
            toks = np.concatenate(recent)
            t.lookup(toks, np.arange(len(recent) + 1, dtype=np.int64) * seq.size, 64)
            t.check_evict()
            if t.gpu.stats()["index_rebuilds"] == 2:
                break
    assert t.gpu.stats()["index_rebuilds"] == 2
    t.check_meta()
    t.close()


def test_rebuild_by_a_small_batch_uses_the_device():
    """An insert of one request that rebuilds the index of 131,072 blocks takes no more than four
    times one that does not (measured: 1.2 times; 19 times when the batch alone sized the grid)."""
    s, g = _full_store(1 << 17)
    for _ in range(30):  # most of a rebuild's worth of deleted slots
        _insert(s, g, 32, 64)
    plain, rebuilding, n = [], [], s.stats()["index_rebuilds"]
    for _ in range(4000):
        us = _insert(s, g, 1, 64)
        now = s.stats()["index_rebuilds"]
        (rebuilding if now > n else plain).append(us)
        if now > n:
            break
        n = now
    s.close()
    assert rebuilding and rebuilding[0] <= 4 * np.median(plain), (rebuilding, np.median(plain))
