"""The autotuner: its choice must count exactly (oracle), a second run of
the same shape must come from the cache, and a fixed placement must be kept."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import to_device
from paper_1607_06618_amd import gerbil as g

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g.load()


def tuned_job(a, o, w, table=g.GERBIL_TABLE_AUTO):
    ad, od = to_device(a, o)
    p = g.make_params(w.k, w.m, w.n_bins, w.threshold, mode=g.GERBIL_BATCHED, table=table)
    job = g.Job(ad, od, int(o[-1]), p, hist_len=512)
    job.encode()
    job.bin()
    info = job.autotune()
    job.count()
    return job, info


def test_autotune_choice_counts_exactly_and_is_cached():
    w = synth.CONFIGS["c2_k65"].scaled(0.004)
    a, o = w.generate()
    ref = oracle.count(a, o, w.k, threshold=w.threshold)
    g.gerbil_autotune_reset()
    job, info = tuned_job(a, o, w)
    assert info.cached == 0 and info.candidates > 0 and info.best_ms > 0
    assert info.table in (g.GERBIL_TABLE_LDS, g.GERBIL_TABLE_HBM)
    assert job.p.table == info.table and job.p.pool == info.pool and job.p.block == info.block
    assert info.block in ((512, 1024) if info.table == g.GERBIL_TABLE_LDS else (256, 512, 1024))
    assert abs(job.p.load_factor - info.load_factor) < 1e-6
    res = job.result()
    keys, counts = res.sorted()
    assert np.array_equal(keys, ref.keys) and np.array_equal(counts, ref.counts)
    assert np.array_equal(res.hist, ref.folded_hist(512))
    # same shape again: the choice comes from the cache, nothing is timed
    job2, info2 = tuned_job(a, o, w)
    assert info2.cached == 1 and info2.candidates == info.candidates
    assert (info2.table, info2.pool, info2.block) == (info.table, info.pool, info.block)
    res2 = job2.result()
    k2, c2 = res2.sorted()
    assert np.array_equal(k2, ref.keys) and np.array_equal(c2, ref.counts)


@pytest.mark.parametrize("table", [g.GERBIL_TABLE_LDS, g.GERBIL_TABLE_HBM])
def test_autotune_keeps_a_fixed_placement(table):
    w = synth.CONFIGS["c1_tiny"].scaled(0.1)
    a, o = w.generate()
    ref = oracle.count(a, o, w.k, threshold=w.threshold)
    g.gerbil_autotune_reset()
    job, info = tuned_job(a, o, w, table=table)
    assert info.table == table and job.p.table == table
    res = job.result()
    keys, counts = res.sorted()
    assert np.array_equal(keys, ref.keys) and np.array_equal(counts, ref.counts)


def long_reads(k, n_reads, seed):
    rng = np.random.default_rng(seed)
    gen = np.array(list(b"ACGT"), np.uint8)[rng.integers(0, 4, 400_000)]
    L = 2 * k + 500
    a = np.concatenate([gen[s:s + L] for s in rng.integers(0, gen.size - L, n_reads).tolist()])
    return a, np.arange(n_reads + 1, dtype=np.uint64) * np.uint64(L)


@pytest.mark.parametrize("mode,k,n_bins", [(g.GERBIL_BATCHED, 300, 16), (g.GERBIL_BATCHED, 479, 64), (g.GERBIL_PLAIN, 55, 256)])
def test_autotune_keeps_the_piece_path(mode, k, n_bins):
    """Keys above 256 bases and the per-bin schedule count by pieces only with AUTO, several times faster than any
    fixed placement: the tuned job keeps it, and counts exactly."""
    a, o = long_reads(k, 4000, k)
    ref = oracle.count(a, o, k, threshold=2)
    g.gerbil_autotune_reset()
    ad, od = to_device(a, o)
    job = g.Job(ad, od, int(o[-1]), g.make_params(k, 9, n_bins, 2, mode=mode), hist_len=512)
    job.encode()
    job.bin()
    info = job.autotune()
    assert info.table == g.GERBIL_TABLE_AUTO and job.p.table == g.GERBIL_TABLE_AUTO
    job.count()
    res = job.result()
    keys, counts = res.sorted()
    assert np.array_equal(keys, ref.keys) and np.array_equal(counts, ref.counts)
    assert np.array_equal(res.hist, ref.folded_hist(512))


def test_autotune_choices_of_other_key_lengths_are_not_shared():
    """k = 17 is partitioned by key hash and k = 31 by pieces: the same key width is not the same shape (one
    bin, of as many k-mers to a quarter octave)."""
    a, o = long_reads(31, 500, 1)
    g.gerbil_autotune_reset()
    ad, od = to_device(a, o)
    for k, cached in ((17, 0), (31, 0), (31, 1)):
        job = g.Job(ad, od, int(o[-1]), g.make_params(k, 9, 1, 1, mode=g.GERBIL_BATCHED), hist_len=512)
        job.encode()
        job.bin()
        assert job.autotune().cached == cached


@pytest.mark.parametrize("mode,k", [(g.GERBIL_PLAIN, 300), (g.GERBIL_PLAIN, 17), (g.GERBIL_BATCHED, 17)])
def test_autotune_names_the_placement_where_auto_is_one(mode, k):
    """Without pieces AUTO is LDS or HBM tables, and the choice says which."""
    a, o = long_reads(k, 300, k)
    g.gerbil_autotune_reset()
    ad, od = to_device(a, o)
    job = g.Job(ad, od, int(o[-1]), g.make_params(k, 9, 16, 1, mode=mode), hist_len=512)
    job.encode()
    job.bin()
    info = job.autotune()
    assert info.table in ((g.GERBIL_TABLE_LDS, g.GERBIL_TABLE_HBM) if k <= 256 else (g.GERBIL_TABLE_HBM,))
    job.count()
    ref = oracle.count(a, o, k, threshold=1)
    keys, counts = job.result().sorted()
    assert np.array_equal(keys, ref.keys) and np.array_equal(counts, ref.counts)
