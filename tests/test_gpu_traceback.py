"""GPU: the traceback's routes against the oracle, word by word, at the sizes
where each can go wrong."""
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
    yield c
    c.close()


def square_pairs(m, n, alphabet, seed):
    """Pairs whose alignment is (nearly always) a square rectangle of about m
    rows: substitutions only in one half, one balanced pair of indels in the
    other, whose diagonal alone scores less than the alignment with gaps."""
    g = np.random.Generator(np.random.PCG64(seed))
    qs, rs = [], []
    for k in range(n):
        core = g.integers(0, alphabet, size=m).astype(np.int8)
        q = core.copy()
        sub = g.random(m) < 0.03
        q[sub] = (q[sub] + 1) % alphabet
        if k % 2 and m >= 24:   # drop a symbol early, add one late
            a, b = m // 3, 2 * m // 3
            q = np.concatenate([q[:a], q[a + 1:b], g.integers(0, alphabet, 1).astype(np.int8), q[b:]])
        left, right = g.integers(0, 20, size=2)
        r = np.concatenate([g.integers(0, alphabet, left), core, g.integers(0, alphabet, right)])
        qs.append(q)
        rs.append(r.astype(np.int8))
    return qs, rs


# the diagonal's sum reads 16-byte words, the last one overlapping
@pytest.mark.parametrize("m", [1, 2, 15, 16, 17, 31, 32, 33, 150, 257])
@pytest.mark.parametrize("alphabet", [4, 24])
def test_main_diagonal_alignments(ctx, m, alphabet):
    qs, rs = square_pairs(m, 96, alphabet, 4000 + m)
    if alphabet == 4:
        b = W.from_lists(f"square-{m}", W.dna_matrix(), 3, 1, qs, rs)
    else:
        b = W.from_lists(f"square-{m}-aa", W.protein_matrix_standin(), 11, 1, qs, rs)
    recs = assert_parity(ctx, b)
    flat = (recs["cigar_len"] == 1)
    assert flat.any()
    assert_parity(ctx, b, flags=swx.SWX_CIGAR)


# a workgroup per pair: strips of 256 rows, one wave each up to four, then in
# turn; the last strip ends with the last row's lane
@pytest.mark.parametrize("m", [1, 3, 4, 5, 255, 256, 257, 512, 700, 1300])
@pytest.mark.parametrize("alphabet", [4, 24])
def test_pair_per_workgroup(ctx, m, alphabet):
    g = np.random.Generator(np.random.PCG64(5000 + m))
    qs, rs = [], []
    for k in range(24):
        core = g.integers(0, alphabet, size=m).astype(np.int8)
        q, _ = W.mutate_many(g, core, np.array([0, m]), 0.05, 0.03, 0.03, 6, alphabet)
        if len(q) == 0 or k % 4 == 3:   # unrelated: weak alignments, wide bands
            q = g.integers(0, alphabet, size=m).astype(np.int8)
        left, right = g.integers(0, 90, size=2)
        r = np.concatenate([g.integers(0, alphabet, left), core, g.integers(0, alphabet, right)])
        qs.append(q)
        rs.append(r.astype(np.int8))
    mat, o, e = (W.dna_matrix(), 3, 1) if alphabet == 4 else (W.protein_matrix_standin(), 11, 1)
    assert_parity(ctx, W.from_lists(f"pairs-{m}-{alphabet}", mat, o, e, qs, rs))


# the routes by scratch size: a few pairs in pair order, a batch by classes,
# and one large enough that only its wide bands go pair by pair
@pytest.mark.parametrize("npairs", [65, 5000, 45000])
def test_traceback_routes_by_batch_size(ctx, npairs):
    b = W.config4(npairs=npairs)
    assert_parity(ctx, b)


# the walk reads 64 cells of a run at a time: runs of matches and gaps around
# that length, gaps behind a run and behind another gap, at both tile sizes
# (long pairs alone spread over workgroups, short strips and tall ones)
@pytest.mark.parametrize("total", [300, 1500, 5000])
@pytest.mark.parametrize("gaps", [(3, 1), (6, 0)])
def test_walk_runs(ctx, total, gaps):
    g = np.random.Generator(np.random.PCG64(6000 + total))
    qs, rs = [], []
    for k in range(12 if total < 5000 else 3):
        q, r = [], []
        while sum(map(len, q)) < total:
            core = g.integers(0, 4, int(g.choice([1, 2, 31, 63, 64, 65, 127, 128, 129])))
            q.append(core)
            r.append(core)
            for side in (q, r) if g.random() < 0.2 else ((q,), (r,))[int(g.integers(0, 2))]:
                side.append(g.integers(0, 4, int(g.choice([1, 1, 1, 2, 3, 63, 64, 65]))))
        qs.append(np.concatenate(q).astype(np.int8))
        rs.append(np.concatenate(r).astype(np.int8))
    assert_parity(ctx, W.from_lists(f"walk-{total}", W.dna_matrix(), *gaps, qs, rs))
