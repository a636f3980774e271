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


@pytest.mark.parametrize("bt,maxb", [(4, 4), (4, 60), (8, 4), (8, 24), (8, 25), (12, 16), (20, 9), (20, 10), (64, 3)])
@pytest.mark.parametrize("R", [4096, 4097])
def test_many_short_requests(R, bt, maxb):
    """Both sides of the rule that takes many requests of few tokens past LDS: more than 4,096
    requests, room for at most 192 tokens each, blocks of four tokens. Stored, cut and fresh
    requests, ragged ends, requests that share their blocks with another of the batch."""
    rng = np.random.default_rng(R + 100 * bt + maxb)
    docs = rng.integers(0, 9, size=(40, maxb * bt), dtype=np.int32)
    rows = []
    for i in range(R):
        d = docs[rng.integers(0, 40)][:int(rng.integers(0, maxb * bt + 1))].copy()
        if d.size and i % 3 == 0:
            d[rng.integers(0, d.size)] += 50 + i % 7
        rows.append(d)
    offs = np.zeros(R + 1, dtype=np.int64)
    offs[1:] = np.cumsum([len(r) for r in rows])
    toks = np.concatenate(rows).astype(np.int32)
    t = Twin(1, 1, 8, bt, 40_000, payload=False)
    t.insert(docs.reshape(-1), np.arange(41, dtype=np.int64) * (maxb * bt), maxb)
    t.lookup(toks, offs, maxb)
    t.insert(toks, offs, maxb)
    t.lookup(toks, offs, maxb)
    t.close()
