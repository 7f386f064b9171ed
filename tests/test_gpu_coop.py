"""GPU: batched tasks shared by the waves of a workgroup, four or (reversed
passes of tall queries) eight, with fewer and more strips than waves."""
from __future__ import annotations

import numpy as np
import pytest

import paper_1208_6350_amd as swx
import workloads as W
from tests.test_gpu_parity import assert_parity

pytestmark = pytest.mark.gpu


# mean query below, at and above eight strips of 32 rows; 130 pairs: two tasks
@pytest.mark.parametrize("qlens", [(200, 255), (256, 257), (250, 520), (600, 700)])
@pytest.mark.parametrize("alphabet", [4, 20])
def test_tall_queries(qlens, alphabet):
    g = np.random.Generator(np.random.PCG64(9000 + qlens[0]))
    qs, rs = [], []
    for k in range(130):
        q = g.integers(0, alphabet, size=int(g.integers(qlens[0], qlens[1] + 1))).astype(np.int8)
        r = g.integers(0, alphabet, size=int(g.integers(100, 500))).astype(np.int8)
        if k % 3:   # a part of the query in the reference, early or late
            n = min(len(q), len(r)) // 2
            at, src = int(g.integers(0, len(r) - n + 1)), int(g.integers(0, len(q) - n + 1))
            r[at:at + n] = q[src:src + n]
        qs.append(q)
        rs.append(r)
    m, gaps = (W.dna_matrix(), (3, 1)) if alphabet == 4 else (W.protein_matrix_standin(), (11, 1))
    c = swx.Context(0)
    c.set_tuning(long_cells=1 << 62, long_rlen=1 << 62, fill_coop=2)
    assert_parity(c, W.from_lists(f"coop-{qlens}-{alphabet}", m, *gaps, qs, rs))
    c.close()


# Tasks whose 128 pairs are copies of one weak pair: a reversed strip near the
# top reaches every target at once and ends, while the strip above it still has
# most of its window to go and the strips below are to end with it.
@pytest.mark.parametrize("qlens", [(120, 250), (260, 400)])   # four and eight waves
@pytest.mark.parametrize("alphabet", [4, 20])
def test_reversed_strips_end_together(qlens, alphabet):
    import oracle
    from tests.fullsize import mismatches

    g = np.random.Generator(np.random.PCG64(9100 + qlens[0] + alphabet))
    copies, kinds = 128, 40
    qs = [g.integers(0, alphabet, size=int(g.integers(qlens[0], qlens[1] + 1))).astype(np.int8)
          for _ in range(kinds)]
    rs = [g.integers(0, alphabet, size=int(g.integers(250, 400))).astype(np.int8) for _ in range(kinds)]
    m, gaps = (W.dna_matrix(), (3, 1)) if alphabet == 4 else (W.protein_matrix_standin(), (11, 1))
    b = W.from_lists("copies", m, *gaps, qs, rs)
    pair = np.repeat(np.arange(kinds), copies)
    ref, rcig, rcoff = oracle.align_many(b.qcat, b.qoff, b.rcat, b.roff, pair, pair, m, *gaps)
    c = swx.Context(0)
    c.set_tuning(long_cells=1 << 62, long_rlen=1 << 62, fill_coop=2)
    for _ in range(3):
        recs, cig = c.align_batch(m, *gaps, b.qcat, b.qoff, b.rcat, b.roff, pair, pair)
        assert mismatches(recs, cig, ref, rcig, rcoff)["pairs_bad"] == 0
    c.close()


# One query against references of very unequal length: the reversed pass on
# eight waves from eight strips of 32 rows on.
@pytest.mark.parametrize("qlen", [255, 256, 257, 520])
def test_search_of_unequal_references(qlen):
    g = np.random.Generator(np.random.PCG64(9200 + qlen))
    q = g.integers(0, 20, size=qlen).astype(np.int8)
    rs = []
    for k in range(130):
        r = g.integers(0, 20, size=1500 if k % 40 == 0 else int(g.integers(60, 300))).astype(np.int8)
        if k % 3:
            n = min(qlen, len(r)) // 2
            at, src = int(g.integers(0, len(r) - n + 1)), int(g.integers(0, qlen - n + 1))
            r[at:at + n] = q[src:src + n]
        rs.append(r)
    b = W.from_lists(f"search-{qlen}", W.protein_matrix_standin(), 11, 1, [q], rs)
    b.pair_q, b.pair_r = np.zeros(len(rs), dtype=np.int64), np.arange(len(rs), dtype=np.int64)
    c = swx.Context(0)
    c.set_tuning(long_cells=1 << 62, long_rlen=1 << 62)
    assert_parity(c, b)
    c.close()
