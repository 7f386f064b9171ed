"""GPU: long pairs whose strips spread over several workgroups (forward,
reversed and traceback), at strip, block and turn boundaries."""
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
    c.set_tuning(long_cells=0, long_rlen=0, intra_bits=32)   # every pair on 32-bit long-pair lanes
    yield c
    c.close()


def long_pairs(qlens, seed, unrelated=False, alphabet=4):
    g = np.random.Generator(np.random.PCG64(seed))
    qs, rs = [], []
    for k, m in enumerate(qlens):
        core = g.integers(0, alphabet, size=m).astype(np.int8)
        q, _ = W.mutate_many(g, core, np.array([0, m]), 0.04, 0.02, 0.02, 4, alphabet)
        if unrelated and k % 2:
            q = g.integers(0, alphabet, size=m).astype(np.int8)
        left, right = g.integers(0, m // 2 + 40, size=2)
        r = np.concatenate([g.integers(0, alphabet, left), core, g.integers(0, alphabet, right)])
        qs.append(q)
        rs.append(r.astype(np.int8))
    return qs, rs


# strips of 128 rows (two per lane) and their edges; blocks of 16 columns
@pytest.mark.parametrize("qlens", [[129], [256, 257], [1024], [1500, 1300, 140], [2600, 300]])
@pytest.mark.parametrize("gaps", [(3, 1), (6, 0), (2, 2)])
def test_spread_dna(ctx, qlens, gaps):
    qs, rs = long_pairs(qlens, 7000 + sum(qlens))
    assert_parity(ctx, W.from_lists(f"spread-{qlens}", W.dna_matrix(), *gaps, qs, rs))


# more strips than waves: each wave takes several in turn; pairs of one shape
def test_spread_turns(ctx):
    qs, rs = long_pairs([900 + 7 * k for k in range(60)], 7100, unrelated=True)
    assert_parity(ctx, W.from_lists("spread-turns", W.dna_matrix(), 3, 1, qs, rs))


def test_spread_protein(ctx):
    qs, rs = long_pairs([700, 1100, 130], 7200, unrelated=True, alphabet=20)
    assert_parity(ctx, W.from_lists("spread-aa", W.protein_matrix_standin(), 11, 1, qs, rs))


# alignments that end in the first strips of the reversed pass, far from the
# corner where its last strips lie
@pytest.mark.parametrize("at", [0, 300, 900])
def test_spread_early_begin(ctx, at):
    g = np.random.Generator(np.random.PCG64(7300 + at))
    q = np.concatenate([np.zeros(at, np.int8), g.integers(0, 4, 200).astype(np.int8),
                        np.full(1000 - at, 1, np.int8)])
    r = np.concatenate([np.full(700, 2, np.int8), q[at:at + 200], np.full(900, 3, np.int8)])
    assert_parity(ctx, W.from_lists(f"spread-early-{at}", W.dna_matrix(), 3, 1, [q, q], [r, r]))
