"""The insert's batch table is empty whenever an insert begins. Inserts of changing batch sizes on
one store, some of them on the exact path, against the CPU oracle, bit-exact."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_22648_amd import ptstore as P
    from tests.twin import Twin


@pytest.mark.parametrize("weak", [False, True])
@pytest.mark.parametrize("evict", [False, True])
def test_batches_of_changing_sizes(evict, weak):
    """One block to several windows a request, tables that grow, shrink and grow again, the same
    prefixes coming back, a store that fills up."""
    rng = np.random.default_rng(3 + evict + 2 * weak)
    flags = (P.PTSTORE_FLAG_EVICT if evict else 0) | (
        P.PTSTORE_FLAG_WEAK_HASH | P.PTSTORE_FLAG_WEAK_TAGS if weak else 0)
    bt = 4
    t = Twin(1, 1, 8, bt, 700, flags=flags, payload=False)
    trunk = rng.integers(0, 9, size=200 * bt, dtype=np.int32)
    for R, maxb in [(3, 5), (40, 150), (1, 1), (7, 64), (64, 65), (2, 200), (40, 150), (5, 130), (90, 3)]:
        reqs = []
        for _ in range(R):
            cut = int(rng.integers(0, maxb + 1)) * bt
            own = rng.integers(0, 9, size=int(rng.integers(0, 6)) * bt + int(rng.integers(0, bt)), dtype=np.int32)
            reqs.append(np.concatenate([trunk[:cut], own]))
        offs = np.zeros(R + 1, dtype=np.int64)
        offs[1:] = np.cumsum([len(r) for r in reqs])
        t.insert(np.concatenate(reqs).astype(np.int32), offs, maxb)
    t.check_meta()
    if evict:
        t.check_evict()
    if weak:
        assert t.gpu.stats()["insert_fallbacks"] >= 1
    t.close()
