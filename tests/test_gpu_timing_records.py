"""ptstore_kernel_times reports the kernels that ran and no others."""
from __future__ import annotations

import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_22648_amd import ptstore as P
    from tests.twin import DEV

BT = 4


def _requests(R, blocks, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    toks = torch.randint(0, 1 << 30, (R * blocks * BT,), dtype=torch.int32, device=DEV, generator=g)
    return toks, torch.arange(R + 1, dtype=torch.int64, device=DEV) * (blocks * BT)


@pytest.mark.parametrize("R", [1, 2])
@pytest.mark.parametrize("layers", [None, (0, 1)])
def test_list_builds_of_a_gather(R, layers):
    """A gather of one request has no list and records no building of one."""
    s = P.PrefixStore(P.StoreShape(2, 1, 8, BT), 100)
    toks, offs = _requests(R, 10, 1)
    m, ids, _ = s.insert(toks, offs, 10)
    table = torch.arange(R * 10, dtype=torch.int32, device=DEV).view(R, 10)
    cache = torch.zeros(R * 10 * s.shape.block_bytes, dtype=torch.uint8, device=DEV)
    s.set_timing(True)
    s.gather(ids, m, table, cache, layers=layers)
    assert s.kernel_times(P.KIND_GATHER)[1] == 1
    assert s.kernel_times(P.KIND_SELECT)[1] == (0 if R == 1 else 1)
    s.close()


@pytest.mark.parametrize("capacity", [16384, 16385])
def test_evictions_of_an_insert(capacity):
    """A store of up to 16,384 blocks evicts inside another of the insert's kernels: no eviction of
    its own to report, only the insert."""
    s = P.PrefixStore(P.StoreShape(1, 1, 8, BT), capacity, flags=P.PTSTORE_FLAG_EVICT)
    s.insert(*_requests(257, 64, 2), 64)
    before = s.stats()["evictions"]
    s.set_timing(True)
    s.insert(*_requests(2, 8, 3), 8)
    assert s.kernel_times(P.KIND_INSERT)[1] == 1
    ms, n = s.kernel_times(P.KIND_EVICT)
    assert (n, ms > 0) == ((0, False) if capacity == 16384 else (1, True))
    assert s.stats()["evictions"] == before + 16
    s.close()
