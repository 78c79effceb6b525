"""Decode options of the LDS-resident decoder with two frames per workgroup
(GPU), whose slots keep an iteration and a test phase each and are refilled one
at a time: every frame against the streaming path, some against the oracle."""
import numpy as np
import pytest

from parity import assert_parity, note, oracle_decode
from test_gpu_lds import CODES, _no_empty, decode, frames

pytestmark = pytest.mark.gpu

# batches that two-frame workgroups take, with more frames than the grid holds
BATCH = {"regular_4096": 700, "regular_4098": 701, "irregular_2600": 2601}


@pytest.mark.parametrize("learned", [False, True])
@pytest.mark.parametrize("L,flags", [(0, 0), (1, 0), (9, 1), (14, 6 << 8), (25, 3 << 8)])
@pytest.mark.parametrize("name", sorted(BATCH))
def test_options(name, L, flags, learned):
    H = _no_empty(CODES[name]())
    llr = frames(H, BATCH[name], seed=17)
    T, C = max(1, L), np.unique(H.sum(1)).size
    rng = np.random.default_rng(6)
    w = (rng.uniform(0.6, 1.1, size=(T, C)).astype(np.float32),
         rng.uniform(0.0, 0.3, size=(T, C)).astype(np.float32)) if learned else ()
    note(f"[lds, two frames] {name} L={L} flags={flags} learned={learned}")
    got = decode(H, llr, L, flags, *w)
    some = np.r_[0:8, len(llr) - 4:len(llr)]  # dealt ones and the last from the counters
    assert_parity(tuple(t[some] for t in got), oracle_decode(H, llr[some], L, flags, *w), name)
