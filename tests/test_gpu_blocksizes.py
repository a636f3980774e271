"""Block sizes by the way their windows are read: sixteen tokens, other multiples of four (through
LDS in parts of sixteen tokens), any other size. Against the CPU oracle, bit-exact."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests.twin import Twin


@pytest.mark.parametrize("maxb", [7, 64, 130, 300])
@pytest.mark.parametrize("bt", [4, 8, 12, 16, 20, 32, 36, 60, 64, 5, 63])
def test_windows_of_any_block(bt, maxb):
    """Requests that start on any token, end inside a block or between two, share prefixes of
    every length (window edges among them) and differ in the first, a middle or the last token
    of one block only; one request has no whole block, one is empty."""
    rng = np.random.default_rng(1000 * bt + maxb)
    root = rng.integers(0, 50, size=maxb * bt, dtype=np.int32)
    docs = [root[:maxb * bt], root[:max(1, maxb // 2) * bt]]
    for cut in sorted({0, 1, maxb // 3, 63, 64, 65, maxb - 1}):
        for at in (0, bt // 2, bt - 1):
            if cut >= maxb:
                continue
            d = root[:min(maxb, cut + 3) * bt].copy()
            d[cut * bt + at] += 77
            docs.append(d)
    reqs = []
    for d in docs:
        for tail in (0, 1, bt - 1):
            reqs.append(np.concatenate([d, rng.integers(0, 50, size=tail, dtype=np.int32)]))
            other = d.copy()
            other[rng.integers(0, len(d))] += 1
            reqs.append(other)
    reqs += [root[:0], root[:bt - 1]]
    order = rng.permutation(len(reqs))
    reqs = [reqs[i] for i in order]

    def pack(rows):
        offs = np.zeros(len(rows) + 1, dtype=np.int64)
        offs[1:] = np.cumsum([len(r) for r in rows])
        return np.concatenate(rows).astype(np.int32), offs

    t = Twin(1, 1, 8, bt, 8192, payload=False)
    t.lookup(*pack(reqs), maxb)
    t.insert(*pack(docs), maxb)
    t.lookup(*pack(reqs), maxb)
    t.insert(*pack(reqs), maxb)
    t.lookup(*pack(reqs), maxb)
    t.check_meta()
    t.close()
