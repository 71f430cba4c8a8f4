"""What this framework is timed on: its public calls, as a program makes them.

The inputs are synthetic metagenome reads made on the GPU (random genomes with
log-normal abundances, reads from both strands, substitution errors, Phred
qualities, some N), with the shapes of the read sets the repository's own
benchmark and tests use.  All results are whole numbers or bytes (tables,
contigs, orders), apart from the two depths a pruning report names.
"""
import ctypes
import math

import numpy as np
import torch

import paper_1809_07014_amd as kh

_COUNT = dict(len_lo=150, len_hi=150, genomes=100, cover=4.3, sigma=1.5, err=0.005, n_rate=0.0,
              min_count=2, bloom=True, shards=0)


def _case(name, kind, reads, ks, **kw):
    return dict(_COUNT, name=name, kind=kind, reads=reads, ks=ks, **kw)


def listed():
    return [
        # one small genome, sequenced deeply: a call bound by its launches
        _case("count_small", "count", 6667, "21", genomes=1, cover=20.0, sigma=0.0, bloom=False),
        # the smallest: a call around graph capture or in a tight loop, no device allocation
        _case("noalloc_small", "noalloc", 1501, "33", genomes=1, cover=20.0, sigma=0.0,
              bloom=False),
        # trimmed reads (ragged lengths, N) of one sample, a higher threshold
        _case("count_ragged", "count", 200_003, "55", len_lo=80, len_hi=250, genomes=20,
              cover=8.0, n_rate=0.002, min_count=3),
        # one sample at one k with the Bloom screen
        _case("count_k31", "count", 2_000_001, "31"),
        # the benchmark's workload: k-mer analysis of 10M reads at every k of the iteration
        _case("multi_k_10M", "count", 10_000_000, "21,33,55,77,99"),
        # one device's part of a key space split over eight
        _case("count_part", "count", 4_000_000, "77", err=0.01, sigma=2.0, genomes=200, shards=8),
        # contigs of one sample's table: the small graph, many short rounds
        _case("traverse_small", "traverse", 100_003, "55", genomes=5),
        # contigs of the large table
        _case("traverse_10M", "traverse", 10_000_000, "21"),
        # contigs of k = 21 join the table at k = 33
        _case("merge_4M", "merge", 4_000_000, "21,33"),
        # Algorithm 2 over the contigs of k = 33
        _case("prune_4M", "prune", 4_000_000, "33"),
        # reads grouped by the contig they come from
        _case("localize_4M", "localize", 4_000_000, "21"),
        # six samples' batches served together from host memory
        _case("serve_6", "serve", 120_000, "21,33,55", genomes=10, bloom=False, samples=6),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def odd(lo, hi):
        return rng.randrange(lo // 2, (hi + 1) // 2) * 2 + 1

    kind = rng.choice(["count"] * 5 + ["noalloc", "traverse", "traverse", "merge", "prune",
                                       "localize", "serve"])
    lo = rng.choice([75, 100, 101, 150, 151, 80])
    hi = lo if lo != 80 else rng.randrange(120, 251)
    c = dict(_COUNT, kind=kind, len_lo=lo, len_hi=hi, genomes=log_int(1, 200),
             cover=rng.choice([3.0, 4.3, 8.0, 20.0]), sigma=rng.choice([0.0, 1.0, 1.5, 2.0]),
             err=rng.choice([0.002, 0.005, 0.01]), n_rate=rng.choice([0.0, 0.0, 0.002]),
             min_count=rng.choice([2, 2, 2, 3]), bloom=rng.random() < 0.7)
    k = odd(15, 71) if hi < 120 else odd(15, 127)
    if kind == "count":
        c.update(reads=log_int(800, 6_000_000), ks=str(k))
        if rng.random() < 0.3:
            c["ks"] = ",".join(str(x) for x in sorted(rng.sample(range(17, 72, 2), 3)))
        elif rng.random() < 0.2:
            c["shards"] = rng.choice([2, 4, 8])
        if not c["bloom"]:
            c["reads"] = min(c["reads"], 2_000_000)
    elif kind == "noalloc":
        c.update(reads=log_int(300, 6_000), ks=str(k), genomes=1, cover=20.0, sigma=0.0,
                 err=min(c["err"], 0.005))
    elif kind == "serve":
        c.update(reads=log_int(5_000, 120_000), ks="21,33,55", bloom=False,
                 samples=rng.randrange(2, 7))
    elif kind == "merge":
        a = odd(19, 31)
        c.update(reads=log_int(10_000, 4_000_000), ks="%d,%d" % (a, a + 2 * rng.randrange(4, 14)))
    else:
        c.update(reads=log_int(10_000, 4_000_000), ks=str(odd(19, 63)))
    return c


# ---- inputs -----------------------------------------------------------------

def _genome_shape(case):
    """Genome lengths (U{2..5} in units that give the wanted coverage), GC and shares of a
    case; what the genomes spell and where the reads lie comes from the seed."""
    rng = np.random.default_rng(1809)
    n = case["genomes"]
    u = rng.uniform(2.0, 5.0, size=n)
    bases = case["reads"] * 0.5 * (case["len_lo"] + case["len_hi"])
    lens = np.maximum(2 * case["len_hi"] + 50, u * bases / case["cover"] / u.sum())
    lens = lens.astype(np.int64)
    w = lens * np.exp(rng.normal(0.0, case["sigma"], size=n))
    return lens, rng.uniform(0.3, 0.7, size=n), w / w.sum()


def _make_reads(case, seed, device="cuda"):
    """(seq, qual, offsets) of one read set, on the GPU, from the seed alone."""
    lens, gc, share = _genome_shape(case)
    sizes = np.random.default_rng(7014).integers(case["len_lo"], case["len_hi"] + 1,
                                                 size=case["reads"])
    g = torch.Generator(device=device)
    g.manual_seed(int(seed) * 7919 + 17)
    parts = []
    for length, p in zip(lens.tolist(), gc.tolist()):  # A C G T = 0 1 2 3
        u = torch.rand(length, generator=g, device=device)
        parts.append((u >= (1 - p) / 2).to(torch.uint8) + (u >= 0.5) + (u >= 1 - (1 - p) / 2))
    genome = torch.cat(parts).to(torch.uint8)
    del parts
    n, lo, hi = case["reads"], case["len_lo"], case["len_hi"]
    gstart = torch.from_numpy(np.concatenate([[0], np.cumsum(lens)[:-1]])).to(device)
    glen = torch.from_numpy(lens).to(device)
    cum = torch.from_numpy(np.cumsum(share)).to(device)
    letters = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device=device)
    seqs, quals, rlens = [], [], []
    col = torch.arange(hi, device=device)
    for r0 in range(0, n, 500_000):
        m = min(500_000, n - r0)
        which = torch.searchsorted(cum, torch.rand(m, generator=g, device=device,
                                                   dtype=torch.float64))
        which.clamp_(max=len(lens) - 1)
        rl = torch.from_numpy(sizes[r0:r0 + m]).to(device)
        room = (glen[which] - rl).double()
        start = (torch.rand(m, generator=g, device=device, dtype=torch.float64) * room).long()
        start += gstart[which]
        back = torch.rand(m, generator=g, device=device) < 0.5
        at = torch.where(back[:, None], rl[:, None] - 1 - col, col.expand(m, hi)).clamp_(min=0)
        b = genome[at.add_(start[:, None]).clamp_(max=genome.numel() - 1)]
        del at
        b = torch.where(back[:, None], 3 - b, b)
        u = torch.rand((m, hi), generator=g, device=device)
        wrong = u < case["err"]
        other = torch.randint(1, 4, (m, hi), generator=g, device=device, dtype=torch.uint8)
        b = torch.where(wrong, (b + other) & 3, b)
        q = torch.randn((m, hi), generator=g, device=device) * 5 + torch.where(wrong, 15.0, 35.0)
        q = q.round_().clamp_(2, 41).to(torch.uint8) + 33
        s = letters[b.long()]
        if case["n_rate"]:
            s = torch.where(u > 1 - case["n_rate"], torch.full_like(s, 78), s)
        keep = (col < rl[:, None])
        seqs.append(s[keep] if lo != hi else s.reshape(-1))
        quals.append(q[keep] if lo != hi else q.reshape(-1))
        rlens.append(rl)
        del b, u, wrong, other, q, s, keep
    off = torch.zeros(n + 1, dtype=torch.int64, device=device)
    torch.cumsum(torch.cat(rlens), 0, out=off[1:])
    return torch.cat(seqs), torch.cat(quals), off


_ctx = {"case": None, "ctx": None}


def _context(case):
    """The program's context; it gives its spare memory back when the work changes."""
    tag = tuple(sorted((k, v) for k, v in case.items() if k != "name"))
    if _ctx["ctx"] is None:
        _ctx["ctx"] = kh.Context(0)
    elif _ctx["case"] != tag:
        _ctx["ctx"].trim()
    _ctx["case"] = tag
    return _ctx["ctx"]


class _HostReads:
    def __init__(self, seq, qual, offsets):
        self.seq, self.qual, self.offsets = (x.cpu().numpy() for x in (seq, qual, offsets))


def _count_args(case):
    return dict(use_bloom=case["bloom"], min_count=case["min_count"],
                owner_shards=case["shards"], owner=0)


def _row_buffers(case, k, many=0, also=0):
    """Room for the rows of a table (and for as many as ``also`` expects) in the program's
    own memory."""
    n = int(1.15 * _expected_rows(case, k)) + 20_000
    n += int(_expected_rows(case, also)) if also else 0
    lead = (many, n) if many else (n,)
    return [torch.zeros(lead + ((k + 31) // 32,), dtype=torch.int64, device="cuda"),
            torch.zeros(lead, dtype=torch.int32, device="cuda"),
            torch.zeros(lead + (8,), dtype=torch.int32, device="cuda"),
            torch.zeros(lead + (2,), dtype=torch.uint8, device="cuda")]


def _contig_buffers(case, k):
    n = int(1.15 * _expected_rows(case, k)) + 20_000
    m = n // 4
    return [torch.zeros(n + m * k, dtype=torch.uint8, device="cuda"),
            torch.zeros(m + 1, dtype=torch.int64, device="cuda"),
            torch.zeros(m, dtype=torch.int64, device="cuda"),
            torch.zeros(m, dtype=torch.int64, device="cuda"),
            torch.zeros(m, dtype=torch.uint8, device="cuda")]


def prepare(case, seed):
    ctx = _context(case)
    ks = [int(x) for x in case["ks"].split(",")]
    st = dict(case=case, ctx=ctx, ks=ks)
    kind = case["kind"]
    if kind == "serve":
        samples = []
        for i in range(case["samples"]):  # each sample's reads come in three batches
            r = _HostReads(*_make_reads(case, seed * 64 + i))
            cut = [0, case["reads"] // 7, case["reads"] // 2, case["reads"]]
            for a, b in zip(cut[:-1], cut[1:]):
                lo, hi = int(r.offsets[a]), int(r.offsets[b])
                part = _HostReads.__new__(_HostReads)
                part.seq, part.qual = r.seq[lo:hi].copy(), r.qual[lo:hi].copy()
                part.offsets = r.offsets[a:b + 1] - lo
                samples.append((i, part))
        samples.sort(key=lambda x: len(x[1].seq))  # batches of the samples arrive mixed
        st.update(batches=samples, server=kh.Server(ks, min_count=case["min_count"]),
                  out=[_row_buffers(case, k, case["samples"]) for k in ks])
        return st
    reads = kh.DeviceReads(*_make_reads(case, seed))
    args = _count_args(case)
    if kind in ("count", "noalloc"):
        st["reads"] = reads
        st["out"] = [_row_buffers(case, k) for k in ks]
        return st
    if kind == "merge":
        st["out"] = _row_buffers(case, ks[1], also=ks[0])
        first, st["table"] = ctx.count_multi_k(reads, ks, **args)
        st["contigs"] = ctx.traverse(first)
        first.free()
        return st
    st["table"] = ctx.count(reads, ks[0], **args)
    if kind in ("traverse", "prune"):
        st["out"] = _contig_buffers(case, ks[0])
    if kind != "traverse":
        st["contigs"] = ctx.traverse(st["table"])
    if kind == "localize":
        st["reads"] = reads
    return st


# ---- the calls --------------------------------------------------------------

def _check(rc):
    if rc:
        raise RuntimeError("kmerhip error %d: %s" % (rc, kh.load().kh_last_error()))


def _export_rows(table, out):
    """The table's rows to the program's buffers (which hold at least as many); freed."""
    inf = table.info()
    n = inf["n_rows"]
    if n > out[1].shape[0]:
        raise RuntimeError("%d rows, room for %d" % (n, out[1].shape[0]))
    _check(kh.load().kh_table_export(table.handle, *[x.data_ptr() for x in out], 1,
                                     torch.cuda.current_stream().cuda_stream))
    table.free()
    return [n, inf["n_windows"]]


def _export_contigs(contigs, out):
    inf = contigs.info()
    if inf["total_bases"] > out[0].shape[0] or inf["n_contigs"] > out[2].shape[0]:
        raise RuntimeError("no room for %s" % inf)
    h = ctypes.c_void_p(contigs._h.value)
    _check(kh.load().kh_contigs_export(h, *[x.data_ptr() for x in out], 1))
    contigs.free()
    return [inf["n_contigs"], inf["total_bases"], inf["cycle_kmers"]]


def run(st):
    case, ctx, ks = st["case"], st["ctx"], st["ks"]
    kind = case["kind"]
    if kind == "count":
        args = _count_args(case)
        if len(ks) == 1:
            tables = [ctx.count(st["reads"], ks[0], **args)]
        else:
            tables = ctx.count_multi_k(st["reads"], ks, **args)
        return [[out, _export_rows(t, out)] for t, out in zip(tables, st["out"])]
    if kind == "noalloc":
        out = st["out"][0]
        return [out, kh.count_noalloc(st["reads"], ks[0], *out, use_bloom=case["bloom"],
                                      min_count=case["min_count"])]
    if kind == "traverse":
        return [st["out"], _export_contigs(ctx.traverse(st["table"]), st["out"])]
    if kind == "merge":
        return [st["out"], _export_rows(ctx.merge_contigs(st["table"], st["contigs"]), st["out"])]
    if kind == "prune":
        kept, rep = ctx.prune(st["table"], st["contigs"])
        return [st["out"], _export_contigs(kept, st["out"]), rep]
    if kind == "localize":
        order = ctx.localize_order(st["table"], st["contigs"], st["reads"])
        r = ctx.gather_reads(st["reads"], order)
        return [order, r.seq, r.qual, r.offsets]
    srv = st["server"]
    tickets = [srv.submit(i, part) for i, part in st["batches"]]
    for t in tickets:
        srv.wait(t)
    sizes = [[_export_rows(t, [x[i] for x in out]) for t, out in zip(srv.finalize(i), st["out"])]
             for i in range(case["samples"])]
    return [st["out"], np.array(sizes)]


# ---- what a pass cannot do without ------------------------------------------

def _expected_rows(case, k):
    """K-mers expected at min_count or more: the genomes' own, and those that one error in
    the same place of several reads makes (3 k per position)."""
    lens, _, share = _genome_shape(case)
    mean = 0.5 * (case["len_lo"] + case["len_hi"])
    windows = case["reads"] * max(0.0, mean - k + 1)
    lam = windows * share / lens * (1 - case["err"]) ** k

    def kept(x):
        return 1 - np.exp(-x) * sum(x ** j / math.factorial(j) for j in range(case["min_count"]))

    once = kept(lam * case["err"] / 3 / (1 - case["err"]))
    rows = float((lens * (kept(lam) + 3 * k * once)).sum())
    return rows / max(1, case["shards"])


def work(case):
    ks = [int(x) for x in case["ks"].split(",")]
    W = [(k + 31) // 32 for k in ks]
    bases = case["reads"] * 0.5 * (case["len_lo"] + case["len_hi"])
    reads = 2 * bases + 8 * case["reads"]
    row = [8 * w + 38 for w in W]
    rows = [_expected_rows(case, k) for k in ks]
    kind = case["kind"]
    if kind in ("count", "noalloc"):
        b = reads + sum(r * n for r, n in zip(row, rows))
    elif kind == "serve":
        b = case["samples"] * (reads + sum(r * n for r, n in zip(row, rows)))
    elif kind == "traverse":  # keys, codes and counts in, one base and its contig out
        b = rows[0] * (8 * W[0] + 6 + 5)
    elif kind == "merge":     # both sets in, the merged rows out
        b = rows[1] * row[1] * 2 + rows[0]
    elif kind == "prune":     # contig bases in and out, the table's row -> contig map
        b = rows[0] * 6
    else:                     # localize: reads in and out, keys looked up once
        b = 2 * reads + 8 * case["reads"] + rows[0] * (8 * W[0] + 4)
    return {"bytes": float(max(b, 1.0)), "flops": 0.0}


def exact(case, seed):
    """Every output is a whole number or a byte, apart from the report's two depths."""
    return None
