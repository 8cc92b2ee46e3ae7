"""The piece partition of the batched counter (bins cut by a second minimizer
into LDS sub-tables) at the key lengths where its layout changes, and on reads
that leave its ordinary path: sub-tables counted in hash slices, strongly
repeated sub-minimizers and piece lists that are too small, both of which the
fallback counts. Exact counts have no tolerance: pairs and histogram equal the
oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
from gpu_util import random_reads, reads_to_csr, to_device
from paper_1607_06618_amd import gerbil as g

pytestmark = pytest.mark.gpu

B = g.GERBIL_BATCHED


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g.load()


def same(res, a, o, k, t, canonical=True):
    ref = oracle.count(a, o, k, threshold=t, canonical=canonical)
    keys, counts = res.sorted()
    assert res.report.n_valid == ref.n_valid
    assert np.array_equal(keys, ref.keys) and np.array_equal(counts, ref.counts)
    assert np.array_equal(res.hist, ref.folded_hist(res.hist.size))


def bases(rng, n):
    return "".join(np.array(list("ACGT"))[rng.integers(0, 4, n)].tolist())


def flip(r):
    return r[::-1].translate(str.maketrans("ACGT", "TGCA"))


def genome_reads(rng, k, glen=6000, n=300, extra=200):
    gen = bases(rng, glen)
    out = []
    for _ in range(n):
        L = int(rng.integers(max(1, k - 3), k + extra))
        s = int(rng.integers(0, glen - L))
        r = gen[s:s + L]
        out.append(flip(r) if rng.random() < 0.5 else r)
    return out + random_reads(rng, 20, 0, k + 60)


# shortest keys; m2 from k/2 to 16; every remainder of the 16-base words; the
# window of middle m2-mers full (k <= 111), then 97 and 96 of them; the longest keys
@pytest.mark.parametrize("canonical", [True, False])
@pytest.mark.parametrize("k", [20, 21, 31, 32, 33, 47, 48, 49, 63, 64, 65, 80, 81, 110, 111, 112, 113, 159, 160, 161,
                               255, 256, 257, 272, 400, 479, 480])
def test_key_lengths(k, canonical):
    rng = np.random.default_rng(900 + 2 * k + canonical)
    a, o = reads_to_csr(genome_reads(rng, k))
    res = g.count_kmers(a, o, k, 9, 13, 1, 64, mode=B, canonical=canonical)
    same(res, a, o, k, 1, canonical)


@pytest.mark.parametrize("block", [512, 1024])
@pytest.mark.parametrize("k,copies", [(31, 40), (65, 30), (65, 120), (65, 900), (200, 60), (200, 700), (300, 500)])
def test_repeated_sub_minimizers(k, copies, block):
    """Reads over one short sequence: few sub-minimizers carry everything, so
    sub-tables are counted whole, in hash slices, or by the fallback."""
    rng = np.random.default_rng(k + copies)
    core = bases(rng, k + 160)
    reads = []
    for i in range(copies):
        r = bases(rng, int(rng.integers(0, 30))) + core + bases(rng, int(rng.integers(0, 30)))
        reads.append(flip(r) if i & 1 else r)
    a, o = reads_to_csr(reads + genome_reads(rng, k, n=60))
    res = g.count_kmers(a, o, k, 9, 4, 1, 2048, mode=B, block=block)
    same(res, a, o, k, 1)


def test_one_window_reads():
    """Every piece is a single k-mer (reads of k and k + 1 bases)."""
    k = 99
    rng = np.random.default_rng(4)
    gen = bases(rng, 5000)
    a, o = reads_to_csr([gen[s:s + k + (s & 1)] for s in rng.integers(0, 4800, 6000).tolist()])
    same(g.count_kmers(a, o, k, 9, 8, 1, 128, mode=B), a, o, k, 1)


@pytest.mark.parametrize("share", [0.35, 0.7])
def test_list_too_small_for_the_pieces(share):
    """A workspace below the one asked for: bins whose pieces do not fit are
    left whole to the fallback, and results stay exact."""
    import torch
    k = 55
    rng = np.random.default_rng(8)
    a, o = reads_to_csr(genome_reads(rng, k, glen=60000, n=6000))
    ad, od = to_device(a, o)
    p = g.make_params(k, 9, 32, 1, mode=B, pool=1, overflow_cap=1 << 12)
    job = g.Job(ad, od, a.size, p, hist_len=128)
    job.encode()
    job.bin()
    job.prepare_count()
    need = job.ws_count.numel()
    fixed = 0   # what a workspace holds besides the pieces: the smallest one that is accepted, to 64 KB
    lo, hi = 0, need
    while hi - lo > 65536:
        mid = (lo + hi) // 2
        st = g.gerbil_count(job.bins, p, job.ws_count.data_ptr(), mid, job.keys_d.data_ptr(), job.counts_d.data_ptr(),
                            job.cap, job.state, g._stream_handle(None))
        lo, hi = (mid, hi) if st == g.GERBIL_EINVAL else (lo, mid)
    torch.cuda.synchronize()
    fixed = hi
    job.ws_count = job.ws_count[: fixed + int(share * (need - fixed)) // 256 * 256]
    job.count()
    same(job.result(), a, o, k, 1)


@pytest.mark.parametrize("n", [1, 63, 65, 255, 257, 1023, 1025, 8200])
@pytest.mark.parametrize("k", [21, 33, 65, 150])
def test_batches_of_super_mers(n, k):
    """One bin whose super-mers end inside, at and past the splitter's batches and items; runs longer than a turn."""
    rng = np.random.default_rng(n * k)
    reads = [bases(rng, k + int(rng.integers(0, 6))) for _ in range(n)] + [bases(rng, 40) + "A" * 400 + bases(rng, 40)]
    a, o = reads_to_csr(reads)
    same(g.count_kmers(a, o, k, 7, 1, 1, 256, mode=B), a, o, k, 1)


@pytest.mark.parametrize("k", [20, 31, 55, 100, 256])
def test_plain_groups(k):
    """PLAIN counts as many bins at a time as the workspace holds: all of them, a few, and one."""
    rng = np.random.default_rng(k)
    a, o = reads_to_csr(genome_reads(rng, k, glen=30000, n=3000))
    ad, od = to_device(a, o)
    p = g.make_params(k, 9, 24, 1, mode=g.GERBIL_PLAIN, overflow_cap=1 << 14)
    job = g.Job(ad, od, a.size, p, hist_len=128)
    job.encode()
    job.bin()
    job.prepare_count()
    need = job.ws_count.numel()

    def count(size):
        return g.gerbil_count(job.bins, p, job.ws_count.data_ptr(), size, job.keys_d.data_ptr(), job.counts_d.data_ptr(),
                              job.cap, job.state, g._stream_handle(None))

    lo, hi = 0, need
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if count(mid) == g.GERBIL_EINVAL else (lo, mid)
    for size in (need, (hi + 3 * need) // 4, (hi + need) // 2, (3 * hi + need) // 4, (15 * hi + need) // 16):
        assert count(size // 256 * 256) == g.GERBIL_OK
        assert g.gerbil_histogram(job.state, job.hist_d.data_ptr(), 128, g._stream_handle(None)) == g.GERBIL_OK
        same(job.result(), a, o, k, 1)


@pytest.mark.parametrize("k,load", [(24, 0.2), (24, 0.06), (24, 0.012), (65, 0.04), (65, 0.01)])
def test_large_bins(k, load):
    """Bins of 500 to 5000 sub-tables: groups of an eighth, a half and a whole
    sub-table, and more of them than the LDS counts take."""
    rng = np.random.default_rng(k)
    a, o = reads_to_csr(genome_reads(rng, k, glen=300000, n=24000))
    same(g.count_kmers(a, o, k, 9, 1, 1, 128, mode=B, load_factor=load), a, o, k, 1)


@pytest.mark.parametrize("k,load,n", [(479, 4.0, 6_000_000), (300, 4.0, 3_000_000), (200, 4.0, 3_000_000)])
def test_sub_tables_cut_by_their_bases(k, load, n):
    """One bin of one long sequence with room for many more k-mers in a sub-table than for their bases: over a
    thousand sub-tables, several times as many as the k-mers would make."""
    rng = np.random.default_rng(k)
    a, o = reads_to_csr([bases(rng, n)])
    same(g.count_kmers(a, o, k, 11, 1, 1, 128, mode=B, load_factor=load), a, o, k, 1)


def test_more_than_a_million_sub_tables_in_a_bin():
    """Weights of a bin's groups that add up to more than 2^32: pairs and histogram as from HBM tables."""
    import torch
    k, n = 65, 72_000_000
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    letters = torch.tensor(list(b"ACGT"), dtype=torch.uint8, device="cuda")
    half = letters[torch.randint(0, 4, (n // 2,), generator=gen, device="cuda")]
    ad = torch.cat([half, half])   # every k-mer but those of the seam twice
    od = torch.tensor([0, n], dtype=torch.int64, device="cuda")
    out = []
    for kw in (dict(table=g.GERBIL_TABLE_HBM), dict(load_factor=0.005)):
        p = g.make_params(k, 9, 1, 2, mode=B, pool=1, **kw)
        job = g.Job(ad, od, n, p, hist_len=16)
        job.run()
        st, rep = g.gerbil_result(job.enc, job.bins, job.state, g._stream_handle(None))
        assert st == g.GERBIL_OK
        keys = job.keys_d[: rep.n_out * job.W].view(-1, job.W)
        out.append((rep.n_out, job.hist_d.cpu().tolist(), keys.sum(0).tolist(), int(job.counts_d[: rep.n_out].sum())))
        del job, keys
    assert out[0] == out[1]
    assert out[0][0] > n // 2 - 2 * k


@pytest.mark.parametrize("k,load", [(65, 4.0), (99, 4.0), (99, 0.0), (200, 0.0)])
def test_large_groups_side_by_side(k, load):
    """One bin whose stretches occur once to 120 times: sub-tables are cut by their bases, from groups of very different sizes."""
    rng = np.random.default_rng(k)
    reads = []
    for _ in range(900):
        s = bases(rng, k + int(rng.integers(20, 300)))
        reads += [s if rng.random() < 0.5 else flip(s) for _ in range(int(120 ** rng.random()))]
    a, o = reads_to_csr([reads[i] for i in rng.permutation(len(reads))])
    same(g.count_kmers(a, o, k, 9, 1, 1, 256, mode=B, load_factor=load), a, o, k, 1)


def test_items_of_a_plain_group_are_of_its_own_super_mers():
    """The split's work items grow with the super-mers of the group (a 2048th of them, or 1024 if a 768th is more than that; 256 to 4096), not with those of
    the bins before it."""
    import torch
    from gpu_util import bin_arrays
    k, n_bins = 41, 64
    rng = np.random.default_rng(5)
    gen = np.array(list(b"ACGT"), np.uint8)[rng.integers(0, 4, 20_000_000)]   # one sequence: about a super-mer for every 17 bases
    o = np.array([0, gen.size], np.uint64)
    ad, od = to_device(gen, o)
    clocks = torch.zeros(8, dtype=torch.int64, device="cuda")
    p = g.make_params(k, 9, n_bins, 1, mode=g.GERBIL_PLAIN, stage_clocks=clocks.data_ptr())
    job = g.Job(ad, od, gen.size, p, hist_len=128)
    job.run()
    job.result()
    _, off, kmers = bin_arrays(job)
    ns, items, groups = np.diff(off.astype(np.int64)), 0, 0
    b = 0
    while b < n_bins:   # groups: bins in order, up to 2^23 k-mers
        e = b + 1
        while e < n_bins and int(kmers[b:e + 1].sum()) <= 1 << 23:
            e += 1
        S = int(ns[b:e].sum())
        descs = min(max((max(S // 2048, min(S // 768, 1024)) + 63) // 64 * 64, 256), 4096)
        items += int((-(-ns[b:e] // descs)).sum())
        groups += 1
        b = e
    assert groups >= 3
    assert int(clocks[4]) == items


@pytest.mark.parametrize("probes", [1, 2, 3, 4, 7, 64])
def test_probes_are_counted_in_slots(probes):
    """max_probes slots, two at a time: no insert ends past that, and the rest takes the emergency area."""
    import torch
    k = 31
    rng = np.random.default_rng(31)
    a, o = reads_to_csr([bases(rng, 300_000)])   # every k-mer once
    ph = torch.zeros(g.GERBIL_PROBE_HIST, dtype=torch.int64, device="cuda")
    res = g.count_kmers(a, o, k, 9, 1, 1, 64, mode=B, load_factor=1.0, max_probes=probes, probe_hist=ph.data_ptr())
    same(res, a, o, k, 1)
    h = ph.tolist()
    most = (probes + 1) // 2
    assert sum(h) == res.report.n_valid
    assert all(x == 0 for x in h[most + 1:-1])
    if probes <= 7:
        assert h[most] > 0 and h[-1] == res.report.n_overflow > 0
