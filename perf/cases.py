"""The alignment work that users of this library have it do, as cases to time.

Each case names a kind of call (below, one class per kind) and its sizes; every
kind goes through a public entry point of paper_1208_6350_amd.  Scoring is the
library's usual: DNA +2/-2 with gap open 3 and extend 1 unless a case says
otherwise, proteins a 24-symbol stand-in matrix with 11/1.  Sequences are
synthetic, drawn from the seed alone, with the error rates of real use: reads
with substitutions and short indels against windows that hold their source,
some of the reads with no source at all, and unrelated database targets.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_1208_6350_amd as swx

DNA, PROTEIN = 4, 24
FLAGS = {"score": 0, "begin": swx.SWX_BEGIN, "cigar": swx.SWX_BEGIN | swx.SWX_CIGAR,
         "all": swx.SWX_ALL, "subopt": swx.SWX_ALL | swx.SWX_SUBOPT}
REC_WORDS = swx.REC_DTYPE.itemsize // 4


@functools.lru_cache(maxsize=1)
def context():
    """The process's one library context: a program makes it once and keeps it."""
    return swx.Context(0)


@functools.lru_cache(maxsize=1)
def protein_scores():
    """A BLOSUM-like stand-in (24 x 24, symmetric, dominant diagonal, expected
    score of two background residues at most -1) and residue frequencies."""
    g = np.random.Generator(np.random.PCG64(24))
    f = g.gamma(4.0, 1.0, size=20)
    f /= f.sum()
    m = g.integers(-4, 4, size=(PROTEIN, PROTEIN))
    m = np.triu(m) + np.triu(m, 1).T
    m[np.arange(PROTEIN), np.arange(PROTEIN)] = g.integers(4, 12, size=PROTEIN)
    off = ~np.eye(20, dtype=bool)
    while f @ m[:20, :20] @ f > -1.0:
        sub = m[:20, :20]
        sub[off] = np.maximum(sub[off] - 1, -4)
        m[:20, :20] = sub
    m[20:, :] = -1
    m[:, 20:] = -1
    return m.astype(np.int8), f


def scoring(case):
    """(matrix, gap open, gap extend) of a case."""
    if case.get("alphabet") == "protein":
        return protein_scores()[0], 11, 1
    m = np.full((DNA, DNA), -2, dtype=np.int8)
    np.fill_diagonal(m, 2)
    return m, case.get("gap_open", 3), case.get("gap_extend", 1)


# ---- sequences ------------------------------------------------------------------
class Draw:
    """Seeded sequences on one device (torch generator of that device)."""

    def __init__(self, seed, device):
        self.dev = torch.device(device)
        self.g = torch.Generator(self.dev).manual_seed(int(seed))

    def ints(self, lo, hi, n):
        return torch.randint(lo, hi, (int(n),), generator=self.g, device=self.dev)

    def unit(self, n):
        return torch.rand(int(n), generator=self.g, device=self.dev)

    def dna(self, n):
        return torch.randint(0, DNA, (int(n),), generator=self.g, device=self.dev,
                             dtype=torch.int8)

    def protein(self, n):
        f = torch.as_tensor(np.cumsum(protein_scores()[1]), device=self.dev, dtype=torch.float32)
        return torch.searchsorted(f, self.unit(n)).clamp_(max=19).to(torch.int8)

    def order(self, n):
        return torch.randperm(n, generator=self.g, device=self.dev).cpu().numpy()

    def mutate(self, cat, lens, sub, ins, dele, max_indel, alphabet=DNA):
        """Substitutions, insertions and deletions (lengths 1..max_indel) at the
        given rates per base, sub one value per sequence or a number.  Returns
        (cat, lens); a sequence never loses its first base."""
        n = cat.numel()
        sid = torch.repeat_interleave(torch.arange(lens.numel(), device=self.dev), lens)
        u = self.unit(n)
        ps = sub[sid] if torch.is_tensor(sub) else torch.full((n,), float(sub), device=self.dev)
        is_sub, is_ins = u < ps, (u >= ps) & (u < ps + ins)
        is_del = (u >= ps + ins) & (u < ps + ins + dele)
        out = torch.where(is_sub, (cat + self.ints(1, alphabet, n)) % alphabet, cat).to(torch.int8)
        run = self.ints(1, max_indel + 1, n)
        keep = torch.ones(n, dtype=torch.bool, device=self.dev)
        start = is_del.nonzero().flatten()
        for t in range(max_indel):
            p = start[run[start] > t] + t
            p = p[p < n]
            p = p[sid[p] == sid[p - t]]
            keep[p] = False
        first = torch.cumsum(lens, 0) - lens
        keep[first] = True
        count = keep * (1 + is_ins * run)
        where = torch.repeat_interleave(torch.arange(n, device=self.dev), count)
        at = torch.cumsum(count, 0) - count
        fresh = torch.arange(where.numel(), device=self.dev) != at[where]
        new = torch.randint(0, alphabet, (where.numel(),), generator=self.g, device=self.dev,
                            dtype=torch.int8)
        lens = torch.zeros_like(lens).scatter_add_(0, sid, count)
        return torch.where(fresh, new, out[where]), lens


def offsets(lens):
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=lens.device)
    off[1:] = torch.cumsum(lens, 0)
    return off


def reads_and_windows(d, n, read_len, flank, sub, indel, max_indel, unrelated):
    """n reads (source lengths read_len = (lo, hi)) and their windows: the
    source plus up to `flank` bases around it.  sub = (lo, hi) per read, indel
    the rate per base, `unrelated` the share of reads with no source."""
    slen = d.ints(read_len[0], read_len[1] + 1, n)
    extra = d.ints(flank[0], flank[1] + 1, n)
    left = (d.unit(n) * (extra + 1)).long().clamp_(max=flank[1])
    left = torch.minimum(left, extra)
    wlen = slen + extra
    roff, soff = offsets(wlen), offsets(slen)
    rcat = d.dna(int(roff[-1]))
    sid = torch.repeat_interleave(torch.arange(n, device=d.dev), slen)
    at = torch.arange(sid.numel(), device=d.dev) - soff[sid] + roff[sid] + left[sid]
    rate = sub[0] + (sub[1] - sub[0]) * d.unit(n)
    qcat, qlen = d.mutate(rcat[at], slen, rate, indel / 2, indel / 2, max_indel)
    qoff = offsets(qlen)
    lone = torch.repeat_interleave(d.unit(n) < unrelated, qlen)
    qcat = torch.where(lone, d.dna(qcat.numel()), qcat)
    idx = torch.arange(n, device=d.dev)
    return qcat, qoff, rcat, roff, idx, idx.clone()


def short_reads(d, n):
    """Reads of a mapper: 100-250 nt, 1-3% substitutions, 0.5% indels, against
    windows with up to 400 nt of flank; 10% of the reads map nowhere."""
    return reads_and_windows(d, n, (100, 250), (0, 400), (0.01, 0.03), 0.005, 3, 0.10)


def cells_of_short_reads(n):
    return n * 67_500.0   # the mean of read length x window length above


def one_pair(case, seed, device):
    """(query, reference) of a single pair, of exactly the case's lengths."""
    d = Draw(seed, device)
    lq, lr = case["qlen"], case["rlen"]
    if case.get("alphabet") == "protein":   # a query against an unrelated target
        return d.protein(lq), d.protein(lr)
    ref = d.dna(lr)
    src_len = min(lr, lq + lq // 8 + 8)
    at = int(d.ints(0, lr - src_len + 1, 1))
    err = case["error"]
    q, _ = d.mutate(ref[at:at + src_len], torch.tensor([src_len], device=d.dev), err / 2,
                    err / 4, err / 4, 3 if err < 0.05 else 1)
    q = torch.cat([q, d.dna(lq)])[:lq]
    for _ in range(case.get("repeats", 0)):   # diverged copies of the locus elsewhere
        c = int(d.ints(0, lr - src_len + 1, 1))
        copy, _ = d.mutate(ref[at:at + src_len], torch.tensor([src_len], device=d.dev), 0.05,
                           0.0, 0.0, 1)
        if abs(c - at) > 2 * src_len:
            ref[c:c + src_len] = copy
    return q.contiguous(), ref


def row_of(words, size):
    """CIGAR numbers in an array of a fixed size, zeros after them."""
    out = np.zeros(size, dtype=np.int64)
    out[:len(words)] = words
    return out


def decoded(case, rec, cigar):
    """A one-pair result as numbers."""
    return {**rec, "cigar": row_of([x for n, op in cigar for x in (n, "MID".index(op))],
                                   case["qlen"] + 64)}


def by_field(recs):
    return {k: np.ascontiguousarray(recs[k]) for k in swx.REC_DTYPE.names}


def words_of(case):
    """CIGAR words that a short-read batch of the case holds at most."""
    return (64 if case["flags"] == "subopt" else 32) * case["pairs"] + 1024


def check(status, what):
    if status != 0:
        raise RuntimeError(f"{what}: {swx.swx_strerror(status)}")


# ---- the kinds of calls -----------------------------------------------------------
class Pair:
    """One read against one window in host memory: profile and alignment in one
    call, as a mapper that refines its hits one by one makes it."""

    @staticmethod
    def prepare(case, seed):
        q, r = (x.numpy() for x in one_pair(case, seed, "cpu"))
        return q, r, scoring(case)

    @staticmethod
    def run(s, case):
        q, r, (m, o, e) = s
        return decoded(case, *context().align_pair(q, r, m, o, e, FLAGS[case["flags"]]))


class Profile:
    """A query's profile made once and kept, aligned against one reference: a
    target in host memory, or one that stays in device memory."""

    @staticmethod
    def prepare(case, seed):
        dev = "cuda" if case["resident"] else "cpu"
        q, r = one_pair(case, seed, dev)
        m, o, e = scoring(case)
        p = Kept(swx.swx_profile_create(context().handle, q.cpu().numpy(), m, o, e))
        return p, (r if case["resident"] else r.numpy())

    @staticmethod
    def run(s, case):
        p, r = s
        flags = FLAGS[case["flags"]]
        if case["resident"]:
            r, flags = (r.data_ptr(), r.numel()), flags | swx.SWX_REF_DEVICE
        return decoded(case, *swx.swx_align(p.handle, r, flags))


class Kept:
    """A profile handle, released with the state that holds it."""

    def __init__(self, handle):
        self.handle = handle

    def __del__(self):
        swx.swx_profile_destroy(self.handle)


class HostBatch:
    """A few reads and windows from host memory, as a mapper hands over one
    bundle of reads."""

    @staticmethod
    def prepare(case, seed):
        return [x.numpy() for x in short_reads(Draw(seed, "cpu"), case["pairs"])], scoring(case)

    @staticmethod
    def run(s, case):
        arrays, (m, o, e) = s
        recs, cigar = context().align_batch(m, o, e, *arrays, flags=FLAGS[case["flags"]])
        return {"recs": by_field(recs), "cigar": row_of(cigar, words_of(case))}


class GraphBatch:
    """Bundles of at most a fixed size through a captured graph: copied in,
    replayed, read back."""

    @staticmethod
    def prepare(case, seed):
        arrays = [x.numpy() for x in short_reads(Draw(seed, "cpu"), case["pairs"])]
        m, o, e = scoring(case)
        cap = case["capacity"]
        g = swx.Graph(context(), m, o, e, cap, 300, 704, cap * 300, cap * 704, cap, cap + 1,
                      flags=FLAGS[case["flags"]], route=1 if case["route"] == "intra" else 0)
        return g, arrays

    @staticmethod
    def run(s, case):
        g, arrays = s
        g.load(*arrays)
        g.run()
        recs, cigar = g.read()
        return {"recs": by_field(recs), "cigar": row_of(cigar, words_of(case))}


class DeviceBatch:
    """Many pairs whose codes and results stay in device memory."""

    @staticmethod
    def outputs(case, n, cigar_words):
        recs = torch.zeros(n * REC_WORDS, dtype=torch.int32, device="cuda")
        sub = torch.zeros_like(recs) if case["flags"] == "subopt" else None
        cigar = torch.zeros(cigar_words, dtype=torch.int32, device="cuda")
        return recs, sub, cigar

    @classmethod
    def prepare(cls, case, seed):
        n = case["pairs"]
        arrays = short_reads(Draw(seed, "cuda"), n)
        return arrays, scoring(case), cls.outputs(case, n, words_of(case))

    @staticmethod
    def run(s, case):
        arrays, (m, o, e), (recs, sub, cigar) = s
        status, used = swx.swx_align_batch(context().handle, m, o, e, *arrays,
                                           flags=FLAGS[case["flags"]],
                                           in_mem=swx.SWX_MEM_DEVICE, recs=recs, cigar=cigar,
                                           out_mem=swx.SWX_MEM_DEVICE, sub_recs=sub)
        check(status, "swx_align_batch")
        out = {"recs": recs, "cigar": cigar, "cigar_used": used}
        return out if sub is None else {**out, "sub_recs": sub}


class ProteinSearch(DeviceBatch):
    """One protein against a database that stays in device memory (target
    lengths LogNormal around 300, clipped to 50-5000)."""

    @classmethod
    def prepare(cls, case, seed):
        d = Draw(seed, "cuda")
        n = case["pairs"]
        z = torch.randn(n, generator=d.g, device=d.dev)
        lens = torch.exp(math.log(300.0) + 0.6 * z).round().clamp_(50, 5000).long()
        roff = offsets(lens)
        q, r = d.protein(case["qlen"]), d.protein(int(roff[-1]))
        # one target in 500 is a relative of the query: 60% of its residues kept
        kin = (d.unit(n) < 0.002).nonzero().flatten()
        m = min(case["qlen"], 50)
        for k in range(m):
            same = d.unit(kin.numel()) < 0.6
            at = roff[kin] + k
            r[at] = torch.where(same, q[k], r[at])
        arrays = (q, torch.tensor([0, case["qlen"]], device="cuda"), r, roff,
                  torch.zeros(n, dtype=torch.int64, device="cuda"),
                  torch.arange(n, device="cuda"))
        return arrays, scoring(case), cls.outputs(case, n, 96 * n + 1024)


class Overlap(DeviceBatch):
    """Every pair of short reads of one region (a read-overlap graph)."""

    @classmethod
    def prepare(cls, case, seed):
        d = Draw(seed, "cuda")
        n, ln, region = case["reads"], case["read_len"], case["region"]
        start = d.ints(0, region - ln + 1, n)
        src = d.dna(region)[(start[:, None] + torch.arange(ln, device="cuda")).flatten()]
        reads, lens = d.mutate(src, torch.full((n,), ln, device="cuda"), 0.01, 0.0, 0.0, 1)
        off = offsets(lens)
        i, j = torch.triu_indices(n, n, 1, device="cuda")
        n = i.numel()
        return (reads, off, reads, off, i.contiguous(), j.contiguous()), scoring(case), \
            cls.outputs(case, n, 32 * n + 1024)


class Serve:
    """A burst of requests to the server, short ones (150-nt reads, 1-kb
    windows) and long ones (10-kb reads at 10% error, 20-kb windows), waited
    for until the last has completed."""

    @staticmethod
    def prepare(case, seed):
        d = Draw(seed, "cpu")
        a = reads_and_windows(d, case["short"], (150, 150), (850, 850), (0.01, 0.01), 0.01, 1, 0.0)
        b = None
        if case["long"]:
            b = reads_and_windows(d, case["long"], (10000, 10000), (10000, 10000), (0.05, 0.05),
                                  0.05, 1, 0.0)
        m, o, e = scoring(case)
        server = swx.Server(m, o, e, mem_budget=32 << 30)
        keep, reqs = [], []
        for k, arrays in enumerate(x for x in (a, b) if x):
            arrays = [x.numpy() for x in arrays]
            n = len(arrays[4])
            base = 0 if k == 0 else case["short"]
            reqs.append(swx.make_requests(*arrays, tags=np.arange(base, base + n)))
            keep.append(arrays)
        reqs = np.concatenate(reqs)
        return server, reqs[d.order(len(reqs))], keep

    @staticmethod
    def run(s, case):
        server, reqs, _ = s
        status, tickets = server.submit(reqs)
        check(status, "swx_server_submit")
        n = len(reqs)
        recs, cigars, got = np.zeros(n, dtype=swx.REC_DTYPE), [None] * n, 0
        while got < n:
            done, cig = server.poll(max_n=n, timeout_us=100000, keep_cigar=True)
            for c, words in zip(done, cig):
                check(int(c["status"]), "request")
                recs[c["tag"]] = c["rec"]
                cigars[c["tag"]] = words
            got += len(done)
        return {"recs": by_field(recs),
                "cigar": row_of(np.concatenate(cigars), 64 * case["short"] + 4096 * case["long"])}


KINDS = {"pair": Pair, "profile": Profile, "host_batch": HostBatch, "graph": GraphBatch,
         "device_batch": DeviceBatch, "protein_search": ProteinSearch, "overlap": Overlap,
         "serve": Serve}


def listed():
    return [
        # the smallest call: one 150-nt read refined against its 2-kb window
        {"name": "pair-dna-150x2000", "kind": "pair", "qlen": 150, "rlen": 2000, "error": 0.025,
         "flags": "all"},
        # one protein against one target, its profile kept: the step of a search
        # that goes target by target
        {"name": "pair-protein-300x350", "kind": "profile", "alphabet": "protein", "qlen": 300,
         "rlen": 350, "error": 0.0, "resident": False, "flags": "all"},
        # one long noisy read against its window
        {"name": "pair-long-10000x20000", "kind": "profile", "qlen": 10000, "rlen": 20000,
         "error": 0.10, "resident": False, "flags": "all"},
        # a 1-kb read against a 5-Mb genome that stays on the device, with
        # diverged copies of its locus (score2 is a real second hit)
        {"name": "genome-1000x5m", "kind": "profile", "qlen": 1000, "rlen": 5_000_000,
         "error": 0.013, "repeats": 3, "resident": True, "flags": "all"},
        # a bundle of reads from host memory, odd in number
        {"name": "reads-host-101", "kind": "host_batch", "pairs": 101, "flags": "all"},
        # the same through a captured graph, fewer reads than its capacity
        {"name": "reads-graph-500of512", "kind": "graph", "pairs": 500, "capacity": 512,
         "route": "intra", "flags": "all"},
        # a device-resident bundle with the suboptimal alignments (mapping quality)
        {"name": "reads-subopt-20k", "kind": "device_batch", "pairs": 20_000, "flags": "subopt"},
        # scores and ends only: a filter over many candidate windows
        {"name": "reads-score-200k", "kind": "device_batch", "pairs": 200_000, "flags": "score"},
        # the benchmark's workload: a million reads, every output
        {"name": "reads-1m", "kind": "device_batch", "pairs": 1_000_000, "flags": "all"},
        # the benchmark's protein search
        {"name": "protein-300x100k", "kind": "protein_search", "alphabet": "protein", "qlen": 300,
         "pairs": 100_000, "flags": "all"},
        # all-vs-all overlap of short reads of one region
        {"name": "overlap-2000x70", "kind": "overlap", "reads": 2000, "read_len": 70,
         "region": 1500, "flags": "all"},
        # a burst at the server, 10% of it long
        {"name": "serve-450+50", "kind": "serve", "short": 450, "long": 50, "flags": "all"},
    ]


def draw(rng):
    def log(lo, hi):   # sizes spread over their logarithm
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["pair", "profile-protein", "profile-long", "genome", "host_batch", "graph",
                       "subopt", "device_batch", "device_batch", "protein_search", "overlap",
                       "serve"])
    gaps = dict(zip(("gap_open", "gap_extend"), rng.choice([(3, 1), (3, 1), (5, 2), (2, 2)])))
    if kind == "pair":
        lr = log(300, 6000)
        return {"kind": "pair", "qlen": min(lr, log(40, 600)), "rlen": lr,
                "error": rng.uniform(0.01, 0.05), "flags": rng.choice(["all", "all", "cigar", "score"]),
                **gaps}
    if kind == "profile-protein":
        return {"kind": "profile", "alphabet": "protein", "qlen": log(60, 1500),
                "rlen": log(50, 5000), "error": 0.0, "resident": rng.random() < 0.3,
                "flags": rng.choice(["all", "all", "begin", "score"])}
    if kind == "profile-long":
        lq = log(1500, 12000)
        return {"kind": "profile", "qlen": lq, "rlen": lq + log(200, 12000),
                "error": rng.uniform(0.02, 0.12), "resident": rng.random() < 0.3, "flags": "all",
                **gaps}
    if kind == "genome":
        return {"kind": "profile", "qlen": log(100, 1000), "rlen": log(100_000, 5_000_000),
                "error": rng.uniform(0.01, 0.03), "repeats": 3, "resident": True, "flags": "all"}
    if kind == "host_batch":
        return {"kind": "host_batch", "pairs": log(2, 3000),
                "flags": rng.choice(["all", "all", "cigar", "begin"]), **gaps}
    if kind == "graph":
        cap = rng.choice([64, 256, 512, 1000])
        return {"kind": "graph", "pairs": rng.randint(cap // 2 + 1, cap), "capacity": cap,
                "route": rng.choice(["intra", "batched"]), "flags": "all", **gaps}
    if kind == "subopt":
        return {"kind": "device_batch", "pairs": log(500, 50_000), "flags": "subopt", **gaps}
    if kind == "device_batch":
        return {"kind": "device_batch", "pairs": log(1000, 600_000),
                "flags": rng.choice(["all", "all", "score", "begin", "cigar"]), **gaps}
    if kind == "protein_search":
        return {"kind": "protein_search", "alphabet": "protein", "qlen": log(60, 600),
                "pairs": log(1000, 100_000), "flags": rng.choice(["all", "all", "score"])}
    if kind == "overlap":
        return {"kind": "overlap", "reads": log(150, 2500), "read_len": rng.randint(50, 100),
                "region": rng.randint(1000, 3000), "flags": "all"}
    long = rng.randint(0, 30)
    return {"kind": "serve", "short": log(20, 1500), "long": long, "flags": "all"}


def prepare(case, seed):
    return case, KINDS[case["kind"]].prepare(case, seed)


def run(state):
    case, s = state
    return KINDS[case["kind"]].run(s, case)


def work(case):
    """Codes in, records and about 8 CIGAR words a pair out; 10 integer
    operations per cell of query x reference (the recurrence and the column
    maximum)."""
    kind = case["kind"]
    if kind in ("pair", "profile"):
        n, cells, codes = 1, case["qlen"] * case["rlen"], case["qlen"] + case["rlen"]
    elif kind == "protein_search":
        n = case["pairs"]
        codes = case["qlen"] + 355 * n   # mean of the target lengths
        cells = case["qlen"] * 355.0 * n
    elif kind == "overlap":
        n = case["reads"] * (case["reads"] - 1) // 2
        codes = case["reads"] * case["read_len"] + 16 * n   # the pair list is an input here
        cells = float(n) * case["read_len"] ** 2
    elif kind == "serve":
        n = case["short"] + case["long"]
        codes = case["short"] * 1150 + case["long"] * 30_000
        cells = case["short"] * 150e3 + case["long"] * 200e6
    else:
        n = case["pairs"]
        codes, cells = 550 * n, cells_of_short_reads(n)
    return {"bytes": float(codes + n * (swx.REC_DTYPE.itemsize + 32)), "flops": 10.0 * cells}


# ---- the same numbers in plain numpy ----------------------------------------------
def _fill(q, r, m, o, e):
    """Local alignment by anti-diagonals in 64 bits.  Returns (column maxima,
    first row reaching each)."""
    lq, lr = len(q), len(r)
    low = -(1 << 40)
    best = np.zeros(lr, dtype=np.int64)
    row = np.full(lr, -1, dtype=np.int64)
    h1 = np.zeros(lq + 1, dtype=np.int64)   # previous anti-diagonal, index i + 1
    h2 = np.zeros(lq + 1, dtype=np.int64)
    ee = np.full(lq + 1, low, dtype=np.int64)
    ff = np.full(lq + 1, low, dtype=np.int64)
    m = m.astype(np.int64)
    for d in range(lq + lr - 1):
        a, b = max(0, d - lr + 1), min(lq - 1, d)
        i = np.arange(a, b + 1)
        j = d - i
        # left neighbour (i, j - 1) and upper (i - 1, j) lie on d - 1
        left_e = np.where(j > 0, ee[a + 1:b + 2], low)
        left_h = np.where(j > 0, h1[a + 1:b + 2], 0)
        up_f = np.where(i > 0, ff[a:b + 1], low)
        up_h = np.where(i > 0, h1[a:b + 1], 0)
        diag = np.where((i > 0) & (j > 0), h2[a:b + 1], 0)
        en = np.maximum(left_e - e, left_h - o)
        fn = np.maximum(up_f - e, up_h - o)
        hn = np.maximum(0, np.maximum(diag + m[q[i], r[j]], np.maximum(en, fn)))
        cur = best[j]
        up = (hn > cur) | ((hn == cur) & (hn > 0) & (i < row[j]))
        best[j] = np.where(up, hn, cur)
        row[j] = np.where(up, i, row[j])
        h2, h1 = h1, np.zeros(lq + 1, dtype=np.int64)
        h1[a + 1:b + 2] = hn
        ee = np.full(lq + 1, low, dtype=np.int64)
        ff = np.full(lq + 1, low, dtype=np.int64)
        ee[a + 1:b + 2] = en
        ff[a + 1:b + 2] = fn
    return best, row


def _alignment(q, r, m, o, e, flags):
    """The documented results of one pair, CIGAR apart: score1, its first end
    (smallest reference, then query position), the begin (largest positions),
    score2 outside the masked columns and its first column."""
    q, r = q.astype(np.int64), r.astype(np.int64)
    best, row = _fill(q, r, m, o, e)
    s1 = int(best.max()) if len(r) else 0
    out = {"score1": s1, "score2": 0, "read_begin1": -1, "read_end1": -1, "ref_begin1": -1,
           "ref_end1": -1, "ref_end2": -1}
    if s1 == 0:
        return out
    je = int(np.argmax(best))
    ie = int(row[je])
    out.update(read_end1=ie, ref_end1=je)
    if flags == 0:
        return out
    rb, rrow = _fill(q[:ie + 1][::-1], r[:je + 1][::-1], m, o, e)
    jb = int(np.argmax(rb == s1))
    out.update(ref_begin1=je - jb, read_begin1=ie - int(rrow[jb]))
    if flags & swx.SWX_SCORE2:
        mask = max(len(q) // 2, 15)
        rest = best.copy()
        rest[max(0, out["ref_begin1"] - mask):je + mask + 1] = 0
        s2 = int(rest.max())
        out.update(score2=s2, ref_end2=int(np.argmax(rest)) if s2 > 0 else -1)
    return out


def exact(case, seed):
    """Scores, ends and begins in 64 bits, where plain numpy takes seconds; the
    CIGAR's layout and the diagnostic lane width have no such value."""
    flags = FLAGS[case["flags"]]
    m, o, e = scoring(case)
    none = {"cigar_off": None, "cigar_len": None, "lane_bits": None}
    if case["kind"] in ("pair", "profile") and case["qlen"] * case["rlen"] <= 3_000_000:
        dev = "cuda" if case.get("resident") else "cpu"
        q, r = (x.cpu().numpy() for x in one_pair(case, seed, dev))
        return {**none, **_alignment(q, r, m, o, e, flags), "cigar": None}
    if case["kind"] == "host_batch" and case["pairs"] <= 200:
        qc, qo, rc, ro, _, _ = (x.numpy() for x in short_reads(Draw(seed, "cpu"), case["pairs"]))
        got = [_alignment(qc[qo[k]:qo[k + 1]], rc[ro[k]:ro[k + 1]], m, o, e, flags)
               for k in range(case["pairs"])]
        kind = {k: swx.REC_DTYPE[k] for k in got[0]}
        return {"recs": {**none, **{k: np.array([g[k] for g in got], dtype=t)
                                    for k, t in kind.items()}}, "cigar": None}
    return None
