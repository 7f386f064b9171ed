"""GPU: the reductions of a long pair's max array (end and score2) at the
lengths where their launch shape changes, with ties across the reference."""
from __future__ import annotations

import numpy as np
import pytest

import paper_1208_6350_amd as swx
import workloads as W
from tests.test_gpu_parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = swx.Context(0)
    c.set_tuning(long_cells=0, long_rlen=0)   # every pair on the intra-sequence path
    yield c
    c.close()


@pytest.mark.parametrize("rlen", [1, 63, 64, 65, 1023, 1024, 1025, 4097, 8191, 8192, 8193, 20000])
def test_end_and_score2_with_ties(ctx, rlen):
    g = np.random.Generator(np.random.PCG64(6000 + rlen))
    qs, rs = [], []
    for k in range(6):
        q = g.integers(0, 4, size=40).astype(np.int8)
        r = g.integers(0, 4, size=rlen - (k % 2 if rlen > 1 else 0)).astype(np.int8)
        # the query itself at several places, first and last columns among
        # them: ties of score1 and of score2
        for at in sorted({0, len(r) // 3, len(r) // 2, len(r) - 40}):
            if 0 <= at and at + 40 <= len(r):
                r[at:at + 40] = q
        qs.append(q)
        rs.append(r)
    qs.append(np.zeros(5, np.int8))          # no positive score
    rs.append(np.full(rlen, 3, np.int8))
    b = W.from_lists(f"ties-{rlen}", W.dna_matrix(), 3, 1, qs, rs)
    assert_parity(ctx, b)
    assert_parity(ctx, b, mask_len=3)
