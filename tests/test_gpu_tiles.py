"""The tile kernel at the edges of its split (every remainder of a window's
length by a thread's 8 positions, the shortest and longest windows, inputs that
end at a tile's edge, runs of several tiles) and both chunk sizes of the
scatter into bins. Super-mers are whole numbers: they equal the oracle's."""
import numpy as np
import pytest

import oracle
from gpu_util import make_job, random_reads, reads_to_csr
from paper_1607_06618_amd import gerbil as g

pytestmark = pytest.mark.gpu

BIG = 1 << 24   # descriptor capacity from which the scatter takes its large chunks


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g.load()


def check(a, o, k, m, nb, order=g.GERBIL_ORDER_KMC2, **kw):
    from gpu_util import bin_arrays
    job = make_job(a, o, k, m=m, n_bins=nb, order=order, **kw)
    job.encode()
    job.bin()
    st, rep = g.gerbil_result(job.enc, job.bins, None)
    assert st == g.GERBIL_OK
    desc, off, km = bin_arrays(job)
    got = np.stack([desc >> np.uint64(24), desc & np.uint64(0xFFFFFF),
                    np.repeat(np.arange(nb, dtype=np.uint64), np.diff(off).astype(np.int64))], 1)
    got = got[np.argsort(got[:, 0], kind="stable")]
    # the oracle's super-mers, cut at the tiles
    sm = oracle.supermers(a, o, k, m, nb, order)
    s, n, b = sm["start"].astype(np.int64), sm["n_kmers"].astype(np.int64), sm["bin"]
    tile = job.bins.tile
    parts = (s + n - 1) // tile - s // tile + 1
    i = np.repeat(np.arange(s.size), parts)
    j = np.arange(i.size) - np.repeat(np.cumsum(parts) - parts, parts)
    lo = np.where(j == 0, s[i], (s[i] // tile + j) * tile)
    hi = np.minimum(s[i] + n[i], (lo // tile + 1) * tile)
    want = np.stack([lo, hi - lo, b[i]], 1).astype(np.uint64)
    assert np.array_equal(got, want)
    assert rep.n_superm == want.shape[0]
    assert np.array_equal(km.astype(np.int64), np.bincount(b, weights=n, minlength=nb).astype(np.int64))


@pytest.mark.parametrize("k,m", [(16, 15), (9, 3), (14, 7), (16, 8)] + [(24 + r, 9) for r in range(9)] +
                         [(72, 9), (73, 9), (480, 15), (480, 2), (480, 1)])
@pytest.mark.parametrize("cap", [0, BIG])
def test_windows(k, m, cap):
    rng = np.random.default_rng(100 * k + m)
    reads = random_reads(rng, 60, 0, 1500, n_rate=0.002, junk="N") + ["AC" * 1500, "T" * 2500]
    a, o = reads_to_csr(reads)
    check(a, o, k, m, 37, superm_cap=cap)


@pytest.mark.parametrize("n", [30, 2047, 2048, 2049, 2048 + 30, 4096, 4097])
def test_ends_at_a_tile(n):
    rng = np.random.default_rng(n)
    a, o = reads_to_csr(random_reads(rng, 1, n, n, n_rate=0.0))
    check(a, o, 30, 8, 5)


@pytest.mark.parametrize("order", [g.GERBIL_ORDER_KMC2, g.GERBIL_ORDER_LEX])
def test_runs_of_tiles(order):
    rng = np.random.default_rng(8)
    a = np.frombuffer(b"ACGT", dtype=np.uint8)[rng.integers(0, 4, 9_000_000)]
    a[rng.integers(0, a.size, 2000)] = ord("N")
    o = np.unique(np.concatenate([[0, a.size], rng.integers(0, a.size, 40_000)])).astype(np.uint64)
    check(a, o, 65, 9, 512, order)
