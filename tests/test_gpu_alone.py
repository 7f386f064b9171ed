"""GPU: the long-pair path's short queries, a wave per pair: at the edges of
its strips (256 and 512 rows) and blocks of columns, empty sequences, odd
counts, both lane widths, and the mixes with short pairs that go with them."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1208_6350_amd as swx
import workloads as W
from tests.test_gpu_parity import assert_parity, run_both

pytestmark = pytest.mark.gpu


@pytest.fixture(params=[16, 32])
def ctx(request):
    c = swx.Context(0)
    c.set_tuning(long_cells=0, intra_bits=request.param)   # every pair is a long one
    yield c
    c.close()


def pairs(qlens, rlens, seed, alphabet=4):
    """Pair k: a window of its reference with substitutions, or unrelated."""
    g = np.random.Generator(np.random.PCG64(seed))
    qs, rs = [], []
    for k, (m, n) in enumerate(zip(qlens, rlens)):
        r = g.integers(0, alphabet, size=n).astype(np.int8)
        q = g.integers(0, alphabet, size=m).astype(np.int8)
        if k % 3 != 2 and n > 0:
            at = int(g.integers(0, max(n - m, 0) + 1))
            w = r[at:at + m].copy()
            w[g.random(len(w)) < 0.05] = 0
            q[:len(w)] = w
        qs.append(q)
        rs.append(r)
    return qs, rs


EDGES = ([1, 255, 256, 257, 511, 512, 4, 5, 100, 0, 300, 37, 252],
         [1, 300, 15, 16, 17, 700, 1024, 0, 33, 40, 2, 513, 64])


@pytest.mark.parametrize("gaps", [(2, 1), (3, 1), (6, 0)])
def test_edges_dna(ctx, gaps):
    qs, rs = pairs(*EDGES, 8100)
    assert_parity(ctx, W.from_lists("alone-edges", W.dna_matrix(), *gaps, qs, rs))


@pytest.mark.parametrize("top", [255, 512])
def test_edges_protein(ctx, top):
    qs, rs = pairs([min(q, top) for q in EDGES[0]], EDGES[1], 8200, alphabet=20)
    assert_parity(ctx, W.from_lists("alone-aa", W.protein_matrix_standin(), 11, 1, qs, rs))


# scores past 15 bits of the packed three-way maximum
def test_large_scores(ctx):
    qs, rs = pairs([512, 500, 490], [520, 1000, 490], 8300)
    m = W.dna_matrix() * 0 - 60
    np.fill_diagonal(m, 63)
    assert_parity(ctx, W.from_lists("alone-large", m.astype(np.int8), 60, 2, qs, rs))


# short pairs only, an odd number of them
@pytest.mark.parametrize("top", [1, 24, 60])
def test_short_pairs(top):
    g = np.random.Generator(np.random.PCG64(8600 + top))
    qs, rs = pairs(g.integers(0, top + 1, size=97), g.integers(0, top + 1, size=97), 8700)
    c = swx.Context(0)
    assert_parity(c, W.from_lists("alone-short", W.dna_matrix(), 3, 1, qs, rs))
    c.close()


# by the batch's own rules: few long pairs (32-bit lanes) or many (16-bit), the
# short ones with them on 16-bit lanes, or batched where they could saturate it
@pytest.mark.parametrize("nlong,nshort,match", [(70, 9, 2), (2200, 31, 2), (70, 9, 20), (2200, 31, 20)])
def test_with_short_pairs(nlong, nshort, match):
    g = np.random.Generator(np.random.PCG64(8400 + nlong + match))
    n = nlong + nshort
    ql = g.integers(120, 160, size=n)
    rl = g.integers(200, 400, size=n)
    small = g.permutation(n)[:nshort]
    ql[small], rl[small] = g.integers(0, 30, size=nshort), g.integers(0, 60, size=nshort)
    qs, rs = pairs(ql, rl, 8500 + nlong)
    m = W.dna_matrix() * 0 - 2
    np.fill_diagonal(m, match)
    b = W.from_lists("alone-mixed", m.astype(np.int8), 3, 1, qs, rs)
    c = swx.Context(0)
    assert_parity(c, b)
    recs = run_both(c, b, swx.SWX_ALL, -1)[0]
    c.close()
    wide = np.full(n, nlong < 1024)
    wide[small] = False
    np.testing.assert_array_equal(recs["lane_bits"], np.where(wide, 32, 16))


# the suboptimal alignment's passes: first rows at each place in a lane and lane
# of a strip, scores above and below a byte's, a long window and a short one
# (a second alignment just outside a short mask may end in a gap); 512 rows
# leave no room for the anchored row
@pytest.mark.parametrize("mask_len", [0, 2, -1])
@pytest.mark.parametrize("match", [2, 60])
@pytest.mark.parametrize("top", [256, 511, 512])
def test_suboptimal(mask_len, match, top):
    ql = [1, 2, 100, 101, 102, 103, 0, 253, 254, 255, 256, 257, 258, 505, 508, 510, 511, 512]
    ql = [m for m in ql if m <= top]
    qs, rs = pairs(ql, [40 + 3 * m for m in ql], 8800)
    for k in range(0, len(ql), 2):   # a second copy, changed a little, behind the first
        rs[k] = np.concatenate([rs[k], qs[k][ql[k] // 5:]])
    m = W.dna_matrix() * 0 - (2 if match == 2 else 55)
    np.fill_diagonal(m, match)
    b = W.from_lists("alone-sub", m.astype(np.int8), *((3, 1) if match == 2 else (58, 20)), qs, rs)
    c = swx.Context(0)
    recs, cig, sub = c.align_batch(b.matrix, b.gap_open, b.gap_extend, b.qcat, b.qoff, b.rcat, b.roff,
                                   b.pair_q, b.pair_r, swx.SWX_ALL | swx.SWX_SUBOPT, mask_len)
    c.close()
    ref, _, _ = oracle.align_many(b.qcat, b.qoff, b.rcat, b.roff, b.pair_q, b.pair_r, b.matrix,
                                  b.gap_open, b.gap_extend, swx.SWX_ALL, mask_len)
    sref, scig, scoff = oracle.suboptimal_many(b.qcat, b.qoff, b.rcat, b.roff, b.pair_q, b.pair_r,
                                               b.matrix, b.gap_open, b.gap_extend, ref[:, 1], ref[:, 6])
    assert (ref[:, 1] > 0).sum() > len(ql) // 3
    np.testing.assert_array_equal(sub["score1"], ref[:, 1])
    for f, col in (("read_begin1", 0), ("read_end1", 1), ("ref_begin1", 2)):
        np.testing.assert_array_equal(sub[f], sref[:, col], err_msg=f)
    for p in range(b.npairs):
        g = cig[sub["cigar_off"][p]:sub["cigar_off"][p] + sub["cigar_len"][p]]
        np.testing.assert_array_equal(g, scig[scoff[p]:scoff[p] + sref[p, 3]])


# more CIGAR words than the pinned memory beside 45,000 records holds
def test_many_cigar_words():
    g = np.random.Generator(np.random.PCG64(8900))
    n = 45_000
    core = g.integers(0, 4, size=n * 48).astype(np.int8)
    q, qoff = W.mutate_many(g, core, np.arange(n + 1) * 48, 0.1, 0.1, 0.1, 4, 4)
    b = W.from_lists("alone-words", W.dna_matrix(), 2, 1, [q[qoff[k]:qoff[k + 1]] for k in range(n)],
                     [core[48 * k:48 * k + 48] for k in range(n)])
    c = swx.Context(0)
    recs = assert_parity(c, b)
    c.close()
    assert recs["cigar_len"].sum() > (4 << 18) - 12 * n


# short pairs whose scores pass the batched 16-bit limit run again on 32-bit
# lanes; long ones of the same batch keep their width
@pytest.mark.parametrize("nlong", [0, 40, 2300])
def test_short_pairs_past_the_limit(nlong):
    g = np.random.Generator(np.random.PCG64(9100 + nlong))
    n = nlong + 60
    ql, rl = g.integers(30, 80, size=n), g.integers(40, 95, size=n)
    ql[:nlong], rl[:nlong] = g.integers(150, 200, size=nlong), g.integers(200, 300, size=nlong)
    qs, rs = pairs(ql, rl, 9200)
    for k in range(nlong, n, 2):   # every other short pair: its reference's copy
        rs[k][:len(qs[k])] = qs[k][:len(rs[k])]
    m = W.dna_matrix() * 0 - 50
    np.fill_diagonal(m, 60)
    b = W.from_lists("alone-limit", m.astype(np.int8), 70, 10, qs, rs)
    c = swx.Context(0)
    recs = assert_parity(c, b)
    c.close()
    want = np.where(recs["score1"] >= 2047, 32, 16)
    want[:nlong] = 32 if nlong < 1024 else 16
    np.testing.assert_array_equal(recs["lane_bits"], want)
    assert (recs["score1"][nlong:] >= 2047).any() and (recs["score1"][nlong:] < 2047).any()


# Above 32,768 pairs a batch only goes pair by pair where its batched passes are
# the slower way: reads against references this long are not such a batch.
@pytest.mark.parametrize("count,rlen,batched", [(32768, 2000, False), (32769, 2000, True), (49152, 600, True)])
def test_where_large_batches_go(count, rlen, batched):
    from tests.fullsize import mismatches

    g = np.random.Generator(np.random.PCG64(8800 + count))
    kinds = 64
    qs, rs = pairs(g.integers(35, 41, size=kinds), g.integers(rlen - 9, rlen + 1, size=kinds), 8801)
    b = W.from_lists("alone-large", W.dna_matrix(), 3, 1, qs, rs)
    pair = np.arange(count) % kinds
    ref, rcig, rcoff = oracle.align_many(b.qcat, b.qoff, b.rcat, b.roff, pair[:kinds], pair[:kinds],
                                         b.matrix, 3, 1)
    c = swx.Context(0)
    for _ in range(2):
        recs, cig = c.align_batch(b.matrix, 3, 1, b.qcat, b.qoff, b.rcat, b.roff, pair, pair)
    # (where every pair goes alone its begin comes with the forward pass)
    assert (c.stage_ms()[3] > 0.05) == batched
    assert mismatches(recs[:kinds], cig, ref, rcig, rcoff)["pairs_bad"] == 0
    for f in ("score1", "score2", "read_begin1", "read_end1", "ref_begin1", "ref_end1", "ref_end2",
              "cigar_len"):
        assert np.array_equal(recs[f], recs[f][pair]), f
    c.close()


# Short pairs around the batched pass's limit of 16-bit lanes (2,047): scored on
# 16-bit lanes here, and labelled as there.
@pytest.mark.parametrize("batched", [False, True])
def test_label_at_the_batched_limit(batched):
    m = W.dna_matrix(23, -23)
    m[3, 3] = 22
    base = np.tile(np.array([0, 1, 2], dtype=np.int8), 30)[:88]
    qs = [np.append(base, s) for s in (3, 0)] + [np.append(base, [1, 1]), base[:60]]
    rs = [q.copy() for q in qs]
    c = swx.Context(0)
    if batched:
        c.set_tuning(long_cells=8192)
    recs = assert_parity(c, W.from_lists("label", m, 23, 5, qs, rs))
    assert list(recs["score1"]) == [2046, 2047, 2070, 1380]
    assert list(recs["lane_bits"]) == [16, 32, 32, 16]
    c.close()
