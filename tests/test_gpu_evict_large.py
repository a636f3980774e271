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
    """An insert of one request that rebuilds the index of 131,072 blocks takes no more than eight
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
    assert rebuilding and rebuilding[0] <= 8 * np.median(plain), (rebuilding, np.median(plain))


def _ranked(prio, depth, ids, n):
    """The n ids that come first by lowest priority, then deepest, then smallest id."""
    order = np.lexsort((ids, -depth, prio))
    return np.sort(ids[order[:n]])


@pytest.mark.parametrize("slots", [1 << 18, 1 << 19])
def test_small_stores_by_index_slots(slots):
    """A store of few blocks in an index of many slots, on both sides of the size that one
    workgroup clears: inserts through a rebuild, each against the oracle."""
    rng = np.random.default_rng(slots)
    t = Twin(1, 1, 8, BT, 16000, index_slots=slots, flags=EVICT, payload=False)
    offs = np.arange(241, dtype=np.int64) * (60 * BT)
    for _ in range(30):
        toks = rng.integers(0, 1 << 30, size=240 * 60 * BT, dtype=np.int32)
        t.insert(toks, offs, 60)
        if t.gpu.stats()["index_rebuilds"]:
            break
    t.lookup(toks, offs, 60)
    t.check_evict()
    assert t.gpu.stats()["index_rebuilds"] == 1
    t.close()


def test_rebuild_of_a_large_index_uses_the_device():
    """An insert into a store of 16,000 blocks that rebuilds an index of 2^24 slots takes no more
    than eight times one that does not (measured: 1.4; 23 when one workgroup cleared it)."""
    s = P.PrefixStore(P.StoreShape(1, 1, 8, BT), 16000, index_slots=1 << 24, flags=EVICT)
    g = torch.Generator(device=DEV)
    g.manual_seed(5)
    s.set_timing(True)
    plain, n = [], 0
    for _ in range(700):
        us = _insert(s, g, 250, 60)
        n = s.stats()["index_rebuilds"]
        if n:
            break
        plain.append(us)
    s.close()
    assert n == 1 and us <= 8 * np.median(plain), (us, np.median(plain))


@pytest.mark.parametrize("bits", [1, 14, 20, 30, 40, 62])
def test_victims_where_one_block_is_much_hotter(bits):
    """All blocks of 600 chains at nearly the same priority but one chain's root, whose priority
    alone takes `bits` bits of the search's key: the digits that tell the others apart come after
    none to all of the search's passes, and in the longest key after all of them. Evictions of a
    few blocks, of more than one pass lists and of most of the store, each against a sort."""
    rng = np.random.default_rng(bits)
    chains, deep = 600, 64
    n = chains * deep
    s = P.PrefixStore(P.StoreShape(1, 1, 8, BT), n, flags=EVICT)
    toks = torch.from_numpy(rng.integers(0, 1 << 30, size=n * BT, dtype=np.int32)).to(DEV)
    s.insert(toks, torch.arange(chains + 1, dtype=torch.int64, device=DEV) * (deep * BT), deep)
    depth = np.tile(np.arange(deep, dtype=np.int64), chains)
    ids = np.arange(n, dtype=np.int64)
    for new in (1, 37, 3000, 30000):
        prio = 5 + rng.integers(0, 2, size=chains, dtype=np.int64).repeat(deep)  # ties, all through
        prio[int(rng.integers(0, chains)) * deep] += 1 << bits
        s.evict_tensors()[1].copy_(torch.from_numpy(prio))
        R = -(-new // 40)
        lens = np.full(R, 40)
        lens[-1] = new - 40 * (R - 1)
        offs = np.concatenate([[0], np.cumsum(lens * BT)]).astype(np.int64)
        t = torch.from_numpy(rng.integers(0, 1 << 30, size=new * BT, dtype=np.int32)).to(DEV)
        m, got, created = s.insert(t, torch.from_numpy(offs).to(DEV), 40)
        assert int(created.sum()) == new
        got, created = got.cpu().numpy(), created.cpu().numpy().astype(bool)
        taken = got[created].astype(np.int64)
        np.testing.assert_array_equal(np.sort(taken), _ranked(prio, depth, ids, new))
        at = np.nonzero(created)  # the new blocks' depths
        depth[got[at]] = at[1]
    s.close()


@pytest.mark.parametrize("bits", [1, 30, 62])
def test_hot_set_where_one_block_is_much_hotter(bits):
    """The same search ranks the host tier for its replicas, by highest priority, then smallest id."""
    rng = np.random.default_rng(bits)
    dev, hostb, reps = 6000, 18000, 2500
    s = P.PrefixStore(P.StoreShape(1, 1, 8, BT), dev + reps, flags=EVICT, host_blocks=hostb,
                      replica_blocks=reps)
    n = dev + hostb
    toks = torch.from_numpy(rng.integers(0, 1 << 30, size=n * BT, dtype=np.int32)).to(DEV)
    s.insert(toks, torch.arange(n // 60 + 1, dtype=torch.int64, device=DEV) * (60 * BT), 60)
    prio = 5 + rng.integers(0, 3, size=n, dtype=np.int64)
    prio[dev + int(rng.integers(0, hostb))] += 1 << bits
    s.evict_tensors()[1].copy_(torch.from_numpy(prio))
    s.replicate()
    have = np.flatnonzero(s.replica_map().cpu().numpy() >= 0)
    np.testing.assert_array_equal(have, _ranked(-prio[dev:], np.zeros(hostb), np.arange(hostb), reps))
    s.close()


def test_one_hot_block_does_not_slow_the_search():
    """Evictions of 128 blocks from 1,048,576 take no more than five times as long when one block's
    priority is 2^20 above the others' as when none is (measured: 1.3 times; 16 times when what two
    passes had left was always one workgroup's)."""
    s, g = _full_store(1 << 20)

    def evict_us():
        us = []
        for _ in range(9):
            s.kernel_times(P.KIND_EVICT)
            _insert(s, g, 2, 64)
            us.append(s.kernel_times(P.KIND_EVICT)[0] * 1e3)
        return float(np.median(us))

    cold = evict_us()
    s.evict_tensors()[1][0] += 1 << 20
    hot = evict_us()
    s.close()
    assert hot <= 5 * cold, (cold, hot)
