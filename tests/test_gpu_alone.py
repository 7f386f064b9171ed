"""GPU: the long-pair path's short queries, a wave per pair: at the edges of
its strips (256 and 512 rows) and blocks of columns, empty sequences, odd
counts, both lane widths, and the mixes with short pairs that go with them."""
from __future__ import annotations

import numpy as np
import pytest

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
