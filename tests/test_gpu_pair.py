"""GPU: the one-pair call (swx_align) against the oracle, at the strip, chunk
and size limits of its short-query kernels, with references on the host and
on the device."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import paper_1208_6350_amd as swx
import workloads as W

pytestmark = pytest.mark.gpu

NAMES = ["score1", "score2", "read_begin1", "read_end1", "ref_begin1", "ref_end1", "ref_end2"]


@pytest.fixture(scope="module")
def ctx():
    c = swx.Context(0)
    yield c
    c.close()


def make_pair(g, qlen, rlen, alphabet, related=True):
    r = g.integers(0, alphabet, size=rlen).astype(np.int8)
    q = g.integers(0, alphabet, size=qlen).astype(np.int8)
    if related and rlen:
        n = min(qlen, rlen)
        at = int(g.integers(0, rlen - n + 1))
        m, _ = W.mutate_many(g, r[at:at + n], np.array([0, n]), 0.05, 0.02, 0.02, 4, alphabet)
        q[:min(len(m), qlen)] = m[:qlen]
    return q, r


def check(rec, cig, q, r, mat, o, e, flags, mask_len=-1):
    a = oracle.align(q, r, mat, o, e, flags, mask_len)
    for f in NAMES:
        want = getattr(a, f)
        if f == "score2" and not flags & swx.SWX_SCORE2:
            want = 0
        if f == "ref_end2" and not flags & swx.SWX_SCORE2:
            want = -1
        if f in ("read_begin1", "ref_begin1") and not flags & 7:
            want = -1
        assert rec[f] == want, (f, rec[f], want, len(q), len(r))
    assert cig == (list(a.cigar) if flags & swx.SWX_CIGAR else [])
    assert rec["lane_bits"] == 32


@pytest.mark.parametrize("qlen", [1, 3, 4, 5, 63, 150, 255, 256, 257, 512, 700, 1025, 2048, 2049])
@pytest.mark.parametrize("rlen", [1, 17, 64, 500, 4100])
def test_sizes(ctx, qlen, rlen):
    g = np.random.Generator(np.random.PCG64(8000 + 7 * qlen + rlen))
    for related in (True, False):
        q, r = make_pair(g, qlen, rlen, 4, related)
        rec, cig = ctx.align_pair(q, r, W.dna_matrix(), 3, 1)
        check(rec, cig, q, r, W.dna_matrix(), 3, 1, swx.SWX_ALL)


@pytest.mark.parametrize("qlen,rlen", [(40, 65535), (150, 65536), (300, 65536), (90, 65537), (0x800, 9000)])
def test_long_references(ctx, qlen, rlen):
    g = np.random.Generator(np.random.PCG64(8100 + qlen))
    q, r = make_pair(g, qlen, rlen, 4)
    rec, cig = ctx.align_pair(q, r, W.dna_matrix(), 3, 1)
    check(rec, cig, q, r, W.dna_matrix(), 3, 1, swx.SWX_ALL)


@pytest.mark.parametrize("gaps", [(1, 1), (2, 2), (5, 2), (4, 0), (0, 0), (40, 3)])
@pytest.mark.parametrize("qlen,rlen", [(100, 900), (300, 700)])
def test_gap_settings(ctx, gaps, qlen, rlen):
    g = np.random.Generator(np.random.PCG64(8200 + qlen + gaps[0]))
    q, r = make_pair(g, qlen, rlen, 4)
    rec, cig = ctx.align_pair(q, r, W.dna_matrix(), *gaps)
    check(rec, cig, q, r, W.dna_matrix(), *gaps, swx.SWX_ALL)


@pytest.mark.parametrize("n", [1, 2, 5, 24, 32])
def test_alphabets_flags_and_masks(ctx, n):
    g = np.random.Generator(np.random.PCG64(8300 + n))
    mat = g.integers(-5, 4, size=(n, n)).astype(np.int8)
    np.fill_diagonal(mat, 6)
    for qlen, rlen in ((120, 300), (600, 400), (1500, 350)):
        q, r = make_pair(g, qlen, rlen, n) if n > 1 else (np.zeros(qlen, np.int8), np.zeros(rlen, np.int8))
        for flags in (0, swx.SWX_BEGIN, swx.SWX_CIGAR, swx.SWX_SCORE2, swx.SWX_ALL):
            rec, cig = ctx.align_pair(q, r, mat, 9, 2, flags, 5)
            check(rec, cig, q, r, mat, 9, 2, flags, 5)


def test_device_references_and_streams(ctx):
    import torch
    g = np.random.Generator(np.random.PCG64(8400))
    s = torch.cuda.Stream()
    for qlen, rlen in ((80, 1000), (500, 900), (3000, 2500), (200, 70001)):
        q, r = make_pair(g, qlen, rlen, 4)
        p = swx.swx_profile_create(ctx.handle, q, W.dna_matrix(), 3, 1)
        big = torch.full((rlen + 9,), 3, dtype=torch.int8, device="cuda")
        big[3:3 + rlen] = torch.from_numpy(r).cuda()   # an unaligned sub-range
        torch.cuda.synchronize()
        for stream in (None, s):
            rec, cig = swx.swx_align(p, (big.data_ptr() + 3, rlen), swx.SWX_ALL | swx.SWX_REF_DEVICE,
                                     -1, stream)
            check(rec, cig, q, r, W.dna_matrix(), 3, 1, swx.SWX_ALL)
        # written by work queued on the caller's stream just before
        with torch.cuda.stream(s):
            late = torch.zeros(rlen, dtype=torch.int8, device="cuda")
            late.copy_(torch.from_numpy(r).pin_memory(), non_blocking=True)
            rec, cig = swx.swx_align(p, (late.data_ptr(), rlen), swx.SWX_ALL | swx.SWX_REF_DEVICE, -1, s)
        check(rec, cig, q, r, W.dna_matrix(), 3, 1, swx.SWX_ALL)
        # pinned host memory passed as a device reference is read through a copy
        pin = torch.from_numpy(r).pin_memory()
        rec, cig = swx.swx_align(p, (pin.data_ptr(), rlen), swx.SWX_ALL | swx.SWX_REF_DEVICE, -1, s)
        check(rec, cig, q, r, W.dna_matrix(), 3, 1, swx.SWX_ALL)
        swx.swx_profile_destroy(p)


def test_bad_symbols_and_empty(ctx):
    import torch
    q = np.arange(50, dtype=np.int8) % 4
    p = swx.swx_profile_create(ctx.handle, q, W.dna_matrix(), 3, 1)
    for bad in (4, 100, -1, -128):
        r = np.zeros(300, np.int8)
        r[177] = bad
        with pytest.raises(swx.SwxError) as err:
            swx.swx_align(p, r)
        assert err.value.status == -1
        with pytest.raises(swx.SwxError) as err:
            t = torch.from_numpy(r).cuda()
            swx.swx_align(p, (t.data_ptr(), 300), swx.SWX_ALL | swx.SWX_REF_DEVICE)
        assert err.value.status == -1
    rec, cig = swx.swx_align(p, np.zeros(0, np.int8))
    assert rec["score1"] == 0 and rec["ref_end1"] == -1 and cig == [] and rec["lane_bits"] == 32
    rec, cig = swx.swx_align(p, q)   # the context still works
    assert rec["score1"] == 100 and cig == [(50, "M")]
    swx.swx_profile_destroy(p)


# Several strips and a warm-up (the widest positive-scoring span) from a small
# part of the reference to nearly all of it, around the last cut that pays, and
# the device memory that the call then keeps.
@pytest.mark.parametrize("qlen,match,ext,rlen", [
    (300, 2, 1, 948), (300, 2, 1, 1024), (300, 2, 1, 1088), (520, 11, 1, 7000), (520, 30, 1, 17000),
    (2048, 11, 1, 65536), (2048, 30, 1, 65536), (2048, 30, 1, 65000)])
def test_warm_ups_and_memory(qlen, match, ext, rlen):
    import torch

    g = np.random.Generator(np.random.PCG64(8600 + qlen + rlen))
    q, r = make_pair(g, qlen, rlen, 4)
    mat = W.dna_matrix(match, -4)
    c = swx.Context(0)
    free = torch.cuda.mem_get_info()[0]
    rec, cig = c.align_pair(q, r, mat, 11, ext, 0)
    held = free - torch.cuda.mem_get_info()[0]
    check(rec, cig, q, r, mat, 11, ext, 0)
    rec, cig = c.align_pair(q, r, mat, 11, ext)
    check(rec, cig, q, r, mat, 11, ext, swx.SWX_ALL)
    c.close()
    assert held <= 160 << 20
