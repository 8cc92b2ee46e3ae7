"""Bins of a few k-mers by key hash: their run sizes come from a sample that holds
all of them, scaled up, and still fit the workspace that was asked for."""
import numpy as np
import pytest

import oracle
from gpu_util import reads_to_csr
from paper_1607_06618_amd import gerbil as g

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g.load()


@pytest.mark.parametrize("table", [g.GERBIL_TABLE_AUTO, g.GERBIL_TABLE_LDS])
@pytest.mark.parametrize("mode", [g.GERBIL_PLAIN, g.GERBIL_BATCHED])
@pytest.mark.parametrize("sample", [0, 1, 2, 32, 500])
def test_bins_of_a_few_k_mers(mode, table, sample):
    rng = np.random.default_rng(sample)
    for k in (4, 12, 19, 31, 132):
        for n_bins in (1, 16, 1024):
            for n in (1, 2, 5, 40):
                a, o = reads_to_csr(["".join(np.array(list("ACGT"))[rng.integers(0, 4, k + int(rng.integers(0, 3)))].tolist())
                                     for _ in range(n)])
                res = g.count_kmers(a, o, k, min(7, k - 1), n_bins, 1, 64, mode=mode, table=table, size_sample=sample)
                ref = oracle.count(a, o, k, threshold=1)
                keys, counts = res.sorted()
                assert np.array_equal(keys, ref.keys) and np.array_equal(counts, ref.counts), (k, n_bins, n)
