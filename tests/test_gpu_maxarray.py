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


# the forward pass of a few long pairs, cut so that the waves number one per
# SIMD: one strip, four pairs of jobs to a workgroup (the last one partly
# filled), or four strips and more; with a reference shorter than the warm-up
# and one that is empty beside them
@pytest.mark.parametrize("bits", [16, 32])
@pytest.mark.parametrize("qlen,rlens", [(30, [9000]), (150, [30001, 700, 5000]), (256, [70000]),
                                        (257, [20000, 20001]), (900, [40000, 0, 1500]),
                                        (1030, [30000])])
def test_planned_chunks(qlen, rlens, bits):
    c = swx.Context(0)
    c.set_tuning(long_cells=0, long_rlen=0, intra_bits=bits)
    g = np.random.Generator(np.random.PCG64(6100 + qlen))
    qs, rs = [], []
    for n in rlens:
        q = g.integers(0, 4, size=qlen).astype(np.int8)
        r = g.integers(0, 4, size=n).astype(np.int8)
        for at in (0, n // 2, n - qlen):   # copies with gaps, their tails reaching the next chunks
            if 0 <= at and at + qlen <= n:
                cp, _ = W.mutate_many(g, q, np.array([0, qlen]), 0.02, 0.01, 0.01, 5)
                r[at:at + min(qlen, len(cp))] = cp[:qlen]
        qs.append(q)
        rs.append(r)
    assert_parity(c, W.from_lists(f"planned-{qlen}", W.dna_matrix(), 3, 1, qs, rs))
    c.close()
