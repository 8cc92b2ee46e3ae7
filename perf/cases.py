"""The work a user of this library has it do, as measurable cases.

A case is a dict of plain values. ``kind`` says which public entry point runs:

  count    reads in device memory -> (k-mer, count) pairs and the count-of-counts
           histogram, through ``gerbil.Job``: encode, bin, count, histogram. ``how``
           is the schedule: "batched" (one persistent run over all bins), "plain"
           (one launch sequence per bin, the default of ``make_params``) or "graph"
           (the batched path captured once and replayed per batch)
  parse    FASTQ or FASTA text -> CSR reads, ``gerbil.parse``
  records  counted pairs -> the binary record stream, ``gerbil.records``
  sketch   HyperLogLog registers of every bin, ``gerbil.hll_registers``

Reads are drawn on the GPU from a seeded genome with diverged repeat copies, from
both strands, with substitution errors and undetermined bases: the shapes of the
workloads in ``synth/`` (1-500 Mbp genomes, 100-250 bp reads or log-normal long
reads, 1-2% errors).
"""
import math

import torch

from paper_1607_06618_amd import gerbil as g

DEV = "cuda"


def _count(name, k, m, bins, t, G, cov, read, **kw):
    c = {"kind": "count", "name": name, "how": "batched", "k": k, "m": m, "bins": bins, "t": t, "G": G, "cov": cov,
         "read": read, "err": 0.01, "rep": 0.05, "canonical": True, "order": "kmc2", "skew": False}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a small plasmid's worth of reads; launches and latency count
        _count("tiny_k32", 32, 7, 64, 2, 20_000, 10.0, 100, rep=0.0),
        # a bacterial-sized batch, captured once and replayed as a serving program does (1 Mbp, 100k x 100 bp)
        _count("bacterium_k32_graph", 32, 7, 64, 2, 1_000_000, 10.0, 100, rep=0.0, how="graph"),
        # an ordinary job of the serving stream: k = 55, 256 bins, 150 bp reads (25 Mbp at 25x)
        _count("job_k55", 55, 9, 256, 2, 25_000_000, 25.0, 150),
        # the headline workload at its full size: 100 Mbp, 30x of 150 bp, k = 65, 512 bins
        _count("genome_k65", 65, 9, 512, 2, 100_000_000, 30.0, 150),
        # a repeat-rich genome under a strongly skewed minimizer -> bin map, k = 99, 250 bp reads
        _count("skewed_k99", 99, 9, 1024, 3, 100_000_000, 20.0, 250, rep=0.15, skew=True),
        # long reads with many errors, k = 200: almost every k-mer is distinct
        _count("longreads_k200", 200, 11, 2048, 2, 60_000_000, 10.0, 0, err=0.02),
        # strand-specific counting (-d) at the paper's smallest k, 101 bp reads
        _count("stranded_k28", 28, 9, 512, 3, 30_000_000, 20.0, 101, canonical=False),
        # the longest keys the library takes (the paper's upper end of k), 15-word keys
        _count("longest_k479", 479, 11, 512, 2, 10_000_000, 10.0, 0, err=0.005),
        # the per-bin schedule, default of make_params and count_kmers
        _count("per_bin_k55", 55, 9, 256, 2, 5_000_000, 25.0, 150, how="plain"),
        # the step before counting: FASTQ text of 6 M reads
        {"kind": "parse", "name": "fastq_text", "format": "fastq", "reads": 6_000_000, "read": 150, "width": 0},
        # the step after counting: 20 M counted pairs to the binary record stream
        {"kind": "records", "name": "records_k65", "k": 65, "pairs": 20_000_000},
        # distinct k-mers of every bin, for sizing tables without counting
        _count("sketch_k65", 65, 9, 512, 2, 20_000_000, 30.0, 150, kind="sketch", regs=12),
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["count"] * 7 + ["parse", "records", "sketch"])
    if kind == "parse":
        fmt = rng.choice(["fastq", "fasta"])
        read = rng.choice([75, 100, 101, 150, 250, rng.randrange(60, 400)])
        return {"kind": "parse", "format": fmt, "reads": _log_uniform(rng, 2_000, 800_000_000 // read), "read": read,
                "width": rng.choice([60, 70, 80, 0]) if fmt == "fasta" else 0}
    if kind == "records":
        k = rng.choice([28, 31, 32, 55, 65, 99, 200, rng.randrange(17, 257)])
        return {"kind": "records", "k": k, "pairs": _log_uniform(rng, 1_000, 800_000_000 // k)}
    how = "batched" if kind == "sketch" else rng.choice(["batched"] * 6 + ["plain", "graph"])
    k = rng.choice([21, 28, 31, 32, 55, 56, 63, 65, 99, 127, 200, rng.randrange(21, 257), rng.randrange(21, 130)])
    if kind == "count" and rng.random() < 0.08:
        k, how = rng.randrange(257, 481), "batched"
    long_reads = k > 120 or rng.random() < 0.15
    read = 0 if long_reads else rng.choice([r for r in (100, 101, 150, 250, rng.randrange(120, 300)) if r >= k + 10] or [300])
    most = 60_000_000 if k > 256 else 300_000_000 if k > 96 else 1_200_000_000
    most = min(most, 120_000_000 if how == "plain" else 300_000_000 if how == "graph" else most)
    bases, cov = _log_uniform(rng, 200_000, most), round(rng.uniform(5, 40), 1)
    order = rng.choice(["kmc2"] * 4 + ["lex", "random"])
    c = _count("", k, rng.choice([7, 9, 9, 10, 11]), rng.choice([64, 256, 512, 1024, rng.randrange(16, 700)]),
               rng.choice([1, 2, 2, 3]), max(5_000, int(bases / cov)), cov, read, how=how, kind=kind,
               err=rng.choice([0.002, 0.01, 0.01, 0.02]), rep=rng.choice([0.0, 0.05, 0.05, 0.15]),
               canonical=rng.random() < 0.85, order=order, skew=order == "kmc2" and rng.random() < 0.15)
    if kind == "sketch":
        c["regs"] = rng.choice([10, 12, 12, 13])
    del c["name"]
    return c


# ------------------------------------------------------------------- inputs

def _generator(seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    return gen


def _genome(G, rep, gen, gc=0.41):
    """Base codes of a genome: random bases, a share `rep` of it copies of other places with 2% substitutions."""
    u = torch.rand(G, generator=gen, device=DEV)
    codes = ((u >= (1 - gc) / 2).to(torch.uint8) + (u >= 0.5).to(torch.uint8) + (u >= 0.5 + gc / 2).to(torch.uint8))
    slot = 5_000   # a copy stays inside a slot of its own
    n = min(int(rep * G / 2_650), G // slot - 1)
    if n > 0:
        ln = torch.randint(300, slot, (n,), generator=gen, device=DEV)
        dst = torch.randperm(G // slot, generator=gen, device=DEV)[:n] * slot
        src = torch.randint(0, G - slot, (n,), generator=gen, device=DEV)
        r = torch.repeat_interleave(torch.arange(n, device=DEV), ln)
        off = torch.arange(r.numel(), device=DEV) - (torch.cumsum(ln, 0) - ln)[r]
        b = codes[src[r] + off]
        sub = torch.rand(r.numel(), generator=gen, device=DEV) < 0.02
        b = torch.where(sub, (b + torch.randint(1, 4, (r.numel(),), generator=gen, device=DEV, dtype=torch.uint8)) & 3, b)
        codes[dst[r] + off] = b
    return codes


def _read_lengths(n, read, G, gen):
    if read:
        return torch.full((n,), min(read, G - 1), dtype=torch.int64, device=DEV)
    # log-normal, median 2000, sigma 0.5, kept to [500, 10000]
    lo, hi = math.log(500 / 2000) / 0.5, math.log(5) / 0.5
    cdf = [0.5 * (1 + math.erf(x / math.sqrt(2))) for x in (lo, hi)]
    u = cdf[0] + (cdf[1] - cdf[0]) * torch.rand(n, generator=gen, device=DEV, dtype=torch.float64)
    z = torch.erfinv(2 * u - 1) * math.sqrt(2)
    return (2000 * torch.exp(0.5 * z)).to(torch.int64).clamp(1, G - 1)


def _n_reads(c):
    mean = c["read"] or 2000 * math.exp(0.125)
    return max(1, math.ceil(c["cov"] * c["G"] / mean))


_CHUNK = 1 << 26   # bases made at a time


def _chunks(offsets):
    """Read ranges of at most about _CHUNK bases: (first read, one past the last)."""
    total, n = int(offsets[-1]), offsets.numel() - 1
    cuts = torch.searchsorted(offsets, torch.arange(0, total + 1, _CHUNK, device=DEV), right=True) - 1
    cuts = sorted(set(cuts.clamp(0, n).tolist()) | {0, n})
    return list(zip(cuts[:-1], cuts[1:]))


def _per_base(offsets, r0, r1):
    """For the bases of reads [r0, r1): their read and their place in it."""
    ln = offsets[r0 + 1:r1 + 1] - offsets[r0:r1]
    r = torch.repeat_interleave(torch.arange(r0, r1, device=DEV), ln)
    return r, torch.arange(int(offsets[r0]), int(offsets[r1]), device=DEV) - offsets[r]


def _reads(c, seed):
    """(ascii uint8 [n_bytes], offsets int64 [n_reads + 1]) on the GPU."""
    gen = _generator(seed)
    codes = _genome(c["G"], c["rep"], gen)
    n = _n_reads(c)
    ln = _read_lengths(n, c["read"], c["G"], gen)
    offsets = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    offsets[1:] = torch.cumsum(ln, 0)
    start = (torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) * (c["G"] - ln + 1)).to(torch.int64)
    back = torch.rand(n, generator=gen, device=DEV) < 0.5
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device=DEV)
    ascii_ = torch.empty(int(offsets[-1]), dtype=torch.uint8, device=DEV)
    for r0, r1 in _chunks(offsets):
        r, off = _per_base(offsets, r0, r1)
        rev = back[r]
        b = codes[start[r] + torch.where(rev, ln[r] - 1 - off, off)]
        b = torch.where(rev, 3 - b, b)
        u = torch.rand(r.numel(), generator=gen, device=DEV)
        turn = torch.randint(1, 4, (r.numel(),), generator=gen, device=DEV, dtype=torch.uint8)
        s = letters[torch.where(u < c["err"], (b + turn) & 3, b).to(torch.int64)]
        s[u > 1 - 0.0005] = ord("N")
        ascii_[int(offsets[r0]):int(offsets[r1])] = s
    return ascii_, offsets


def _digits(v):
    """How many decimal digits each value has."""
    n = torch.ones_like(v)
    for e in range(1, 12):
        n += v >= 10 ** e
    return n


def _headers(text, at, lead, ids):
    """Write `lead`, the decimal id and a newline at text[at] of every record; returns the headers' lengths."""
    nd = _digits(ids)
    for j, ch in enumerate(lead):
        text[at + j] = ch
    for j in range(12):
        sel = nd > j
        if not bool(sel.any()):
            break
        power = torch.pow(torch.tensor(10, device=DEV), nd[sel] - 1 - j)
        text[at[sel] + len(lead) + j] = (48 + (ids[sel] // power) % 10).to(torch.uint8)
    text[at + len(lead) + nd] = 10
    return nd + len(lead) + 1


def _text(c, seed):
    """FASTQ (random qualities) or FASTA text of c["reads"] reads as a uint8 tensor on the GPU."""
    rc = {"G": max(5_000, c["reads"] * c["read"] // 20), "rep": 0.05, "cov": 0.0, "read": c["read"], "err": 0.01}
    rc["cov"] = c["reads"] * c["read"] / rc["G"]
    ascii_, offsets = _reads(rc, seed)
    n = offsets.numel() - 1
    gen = _generator(seed + 1)
    ids = torch.arange(n, device=DEV)
    ln = offsets[1:] - offsets[:-1]
    lead = list(b"@SYN.") if c["format"] == "fastq" else list(b">syn_")
    head = _digits(ids) + len(lead) + 1
    width = c["width"] or 1 << 30
    rec = head + (2 * ln + 4 if c["format"] == "fastq" else ln + (ln + width - 1) // width)
    at = torch.cumsum(rec, 0) - rec
    text = torch.full((int(rec.sum()),), 10, dtype=torch.uint8, device=DEV)   # every byte not written below ends a line
    _headers(text, at, lead, ids)
    for r0, r1 in _chunks(offsets):
        r, off = _per_base(offsets, r0, r1)
        p = at[r] + head[r] + off
        text[p if c["format"] == "fastq" else p + off // width] = ascii_[int(offsets[r0]):int(offsets[r1])]
        if c["format"] == "fastq":
            text[p + ln[r] + 3] = torch.randint(33, 75, (r.numel(),), generator=gen, device=DEV, dtype=torch.uint8)
    if c["format"] == "fastq":
        text[at + head + ln + 1] = ord("+")
    return text


def _bin_map(c, seed):
    """Minimizer code -> bin with log-normal bin weights."""
    gen = _generator(seed + 2)
    cdf = torch.cumsum(torch.exp(0.97 * torch.randn(c["bins"], generator=gen, device=DEV, dtype=torch.float64)), 0)
    u = torch.rand(4 ** c["m"], generator=gen, device=DEV, dtype=torch.float64)
    return torch.searchsorted(cdf / cdf[-1], u).clamp(0, c["bins"] - 1).to(torch.int32)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "parse":
        return {"kind": kind, "text": _text(case, seed)}
    if kind == "records":
        gen, W = _generator(seed), g.words(case["k"])
        keys = torch.randint(-2 ** 63, 2 ** 63 - 1, (case["pairs"], W), generator=gen, device=DEV)
        r = case["k"] - 32 * (W - 1)
        if r < 32:
            keys[:, W - 1] &= (1 << (2 * r)) - 1
        # counts around the coverage, one in a thousand from a repeat (and stored in the long form)
        counts = 2 + torch.poisson(torch.full((case["pairs"],), 12.0, device=DEV), generator=gen).to(torch.int32)
        many = torch.randperm(case["pairs"], generator=gen, device=DEV)[: case["pairs"] // 1000]
        counts[many] = 255 + 100 * counts[many]
        return {"kind": kind, "keys": keys, "counts": counts, "n": case["pairs"], "k": case["k"]}
    ascii_, offsets = _reads(case, seed)
    keep = []
    kw = {"mode": g.GERBIL_PLAIN if case["how"] == "plain" else g.GERBIL_BATCHED, "canonical": case["canonical"]}
    if case["order"] == "lex":
        kw["order"] = g.GERBIL_ORDER_LEX
    if case["order"] == "random":
        keep.append(g.order_table(g.GERBIL_RANKS_RANDOM, case["m"], seed=seed))
        kw.update(order=g.GERBIL_ORDER_TABLE, rank_table_ptr=keep[-1].data_ptr())
    if case["skew"]:
        keep.append(_bin_map(case, seed))
        kw["bin_map_ptr"] = keep[-1].data_ptr()
    params = g.make_params(case["k"], case["m"], case["bins"], case["t"], **kw)
    stream = torch.cuda.Stream() if case["how"] == "graph" else None   # capture needs a stream of its own
    if stream is not None:
        stream.wait_stream(torch.cuda.current_stream())
    job = g.Job(ascii_, offsets, ascii_.numel(), params, cap=_capacity(case), stream=stream)
    job.encode()
    job.bin()
    if kind == "sketch":
        return {"kind": kind, "job": job, "regs": case["regs"], "keep": keep}
    job.prepare_count()   # workspace and output arrays, sized once for inputs of this shape
    if case["how"] == "graph":
        job.capture()
    return {"kind": kind, "job": job, "keep": keep, "replay": case["how"] == "graph"}


class Counted(dict):
    """Outputs of a counting pass: every pair (zeros after the last, up to the job's
    capacity), the histogram and the report's counts.

    The library emits pairs in no particular order (include/gerbil.h), so whoever
    compares two passes has to order them: they are put in key order here when they
    are read. Nothing of the pass itself waits for that."""

    def __init__(self, job):
        super().__init__(dict.fromkeys(("keys", "counts", "hist", "n_valid", "max_count")))
        self.job, self.read = job, False

    def __getitem__(self, name):
        if not self.read:
            job = self.job
            st, rep = g.gerbil_result(job.enc, job.bins, job.state, g._stream_handle(job.stream))
            if st != g.GERBIL_OK:
                raise g.GerbilError("gerbil_result", st, rep)
            keys = job.keys_d[: rep.n_out * job.W].view(-1, job.W)
            place = torch.arange(rep.n_out, device=DEV)
            for w in reversed(range(job.W)):   # stable, last word first; the flipped sign bit makes the order unsigned
                place = place[torch.sort(keys[place, w] ^ (-2 ** 63), stable=True)[1]]
            out_k, out_c = torch.zeros((job.cap, job.W), dtype=torch.int64, device=DEV), torch.zeros_like(job.counts_d)
            out_k[: rep.n_out], out_c[: rep.n_out] = keys[place], job.counts_d[: rep.n_out][place]
            self.update(keys=out_k, counts=out_c, hist=job.hist_d, n_valid=rep.n_valid, max_count=rep.max_count)
            self.read = True
        return super().__getitem__(name)


def run(state):
    if state["kind"] == "parse":
        p = g.parse(state["text"])
        return {"seq": p.seq, "offsets": p.offsets, "lines": p.info.n_lines, "status": p.info.status}
    if state["kind"] == "records":
        return g.records(state["keys"], state["counts"], state["n"], state["k"])
    if state["kind"] == "sketch":
        return g.hll_registers(state["job"], state["regs"])
    if state["replay"]:
        state["job"].replay()
    else:
        state["job"].run()
    return Counted(state["job"])


def exact(case, seed):
    # every output is a byte or a whole number: equal, or wrong
    return None


def _pairs(c):
    """About how many pairs a counting case emits: a Poisson number of error-free occurrences per genome position."""
    mean = c["read"] or 2000 * math.exp(0.125)
    each = c["cov"] * max(0.0, mean - c["k"] + 1) / mean
    strands = 1 if c["canonical"] else 2
    each /= strands
    clean = each * (1 - c["err"]) ** c["k"]
    under = sum(math.exp(-clean) * clean ** i / math.factorial(i) for i in range(c["t"]))
    return c["G"] * strands * (1 - under + (each - clean if c["t"] == 1 else 0))


def _capacity(c):
    """Output capacity of a counting job, in pairs: what such a program expects, and some room."""
    return int(1.3 * _pairs(c)) + 4096


def work(case):
    if case["kind"] == "parse":
        bases = case["reads"] * case["read"]
        text = bases * (2 if case["format"] == "fastq" else 1) + 16 * case["reads"]
        return {"bytes": text + bases + 8 * case["reads"], "flops": 0}
    if case["kind"] == "records":
        return {"bytes": case["pairs"] * (8 * g.words(case["k"]) + 4 + 1 + (case["k"] + 3) // 4), "flops": 0}
    bases = case["cov"] * case["G"]
    if case["kind"] == "sketch":   # packed bases of the super-mers and their descriptors in, registers out
        return {"bytes": bases / 4 + 8 * bases / 40 + 4 * (case["bins"] << case["regs"]), "flops": 0}
    return {"bytes": bases + 8 * _n_reads(case) + _pairs(case) * (8 * g.words(case["k"]) + 4) + 2048, "flops": 0}
