"""The sketch kernel where its split into segments changes: every way a key
ends in its last half word, the longest keys, super-mers of whole tiles (more
segments than a wave lists at a time), single windows and the largest and
smallest register arrays. Registers are whole numbers: they equal those built
on the host from the emitted keys."""
import numpy as np
import pytest

from gpu_util import make_job, random_reads, reads_to_csr
from paper_1607_06618_amd import gerbil as g
from test_gpu_orders import _bit_length, _key_hash

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g.load()


@pytest.mark.parametrize("k,p", [(10, 10), (16, 4), (17, 12), (32, 10), (33, 13), (47, 10), (48, 15), (49, 10), (97, 10),
                                 (98, 12), (112, 10), (129, 10), (256, 10), (257, 12), (479, 10), (480, 11)])
@pytest.mark.parametrize("canonical", [True, False])
def test_registers(k, p, canonical):
    rng = np.random.default_rng(k)
    reads = (random_reads(rng, 150, k, k + 400, n_rate=0.002, junk="N") + random_reads(rng, 70, k, k, n_rate=0.0) +
             ["A" * 5000, "AC" * 2500, "T" * (k + 2100)])
    a, o = reads_to_csr(reads)
    nb = 7
    job = make_job(a, o, k, m=9, n_bins=nb, threshold=1, mode=g.GERBIL_BATCHED, canonical=canonical)
    job.run()
    res = job.result()
    n = res.counts.size
    bins = g.key_bins(job.keys_d, n, job.p).cpu().numpy().astype(np.int64)
    regs = g.hll_registers(job, p).cpu().numpy()
    h = _key_hash(res.keys.astype(np.uint64), 0x5BD1E9955BD1E995)
    idx = (h >> np.uint64(64 - p)).astype(np.int64)
    rho = 64 - _bit_length((h << np.uint64(p)) | np.uint64(1 << (p - 1))) + 1
    want = np.zeros((nb, 1 << p), dtype=np.int64)
    np.maximum.at(want, (bins, idx), rho)
    assert np.array_equal(regs.astype(np.int64), want)
