"""Requests whose blocks fill a whole round of the lookup's parallel windows (256, 512 and 1,024
blocks at 4, 8 and 16 waves), every one of them stored, with index keys that collide. Against the
CPU oracle, bit-exact."""
from __future__ import annotations

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2607_22648_amd import ptstore as P
    from tests.twin import Twin


@pytest.mark.parametrize("bt", [4, 5, 16])
@pytest.mark.parametrize("maxb", [256, 512, 1024, 1300, 2048])
def test_stored_requests_that_fill_a_round(maxb, bt):
    """Three distinct blocks make up every request and index keys have 8 bits, so lanes find their
    tokens under another parent and probe on. Once the last such lane of a round has found its
    block no position of the round fails any more, and the match goes on to the request's end: a
    lookup returns it whole and an insert of the same requests adds nothing."""
    rng = np.random.default_rng(7 * maxb + bt)
    atoms = rng.integers(0, 32000, size=(3, bt), dtype=np.int32)
    R = 6
    toks = atoms[rng.integers(0, 3, size=R * maxb)].reshape(-1)
    offs = np.arange(R + 1, dtype=np.int64) * (maxb * bt)
    t = Twin(1, 1, 8, bt, 40_000, flags=P.PTSTORE_FLAG_WEAK_HASH, payload=False)
    t.insert(toks, offs, maxb)
    stored = t.ref.count
    (m, _), (rm, _) = t.lookup(toks, offs, maxb)
    assert (rm == maxb).all()
    t.insert(toks, offs, maxb)
    assert t.ref.count == stored
    # the same requests cut inside a round, at its edge and past it
    cuts = [1, maxb // 2, maxb - 1, maxb, min(maxb, 256), min(maxb, 1024)]
    part = np.concatenate([toks[offs[i]:offs[i] + c * bt] for i, c in enumerate(cuts)])
    poffs = np.concatenate([[0], np.cumsum([c * bt for c in cuts])]).astype(np.int64)
    t.lookup(part, poffs, maxb)
    t.check_meta()
    t.close()
