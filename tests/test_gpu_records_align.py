"""The record writer at output addresses that are not multiples of 16 bytes,
with every remainder of a key's bytes by a word, and at capacities that end
inside a 16-byte word: the oracle's bytes, and nothing before or after them."""
import numpy as np
import pytest

from paper_1607_06618_amd import gerbil as g
from test_gpu_records import device_pairs, oracle_stream, random_pairs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g.load()


@pytest.mark.parametrize("k", [1, 8, 9, 13, 20, 32, 33, 70, 76, 82, 257, 480])
@pytest.mark.parametrize("shift,short", [(0, 0), (1, 0), (7, 3), (15, 16), (8, 1)])
def test_output_address(k, shift, short):
    import torch
    rng = np.random.default_rng(k)
    n = 2100
    keys, counts = random_pairs(rng, n, k)
    kd, cd = device_pairs(keys, counts)
    ref = oracle_stream(keys, counts, k)
    cap = len(ref) - short
    ws = torch.empty(g.gerbil_records_workspace(n), dtype=torch.uint8, device="cuda")
    out = torch.full((len(ref) + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    size = torch.zeros(1, dtype=torch.int64, device="cuda")
    st = g.gerbil_records(kd.data_ptr(), cd.data_ptr(), n, k, ws.data_ptr(), ws.numel(), out.data_ptr() + shift, cap,
                          size.data_ptr(), int(torch.cuda.current_stream().cuda_stream))
    assert st == g.GERBIL_OK
    torch.cuda.synchronize()
    assert int(size.item()) == len(ref)
    host = out.cpu().numpy().tobytes()
    assert host[shift: shift + cap] == ref[:cap]
    assert host[:shift] == b"\xa5" * shift and host[shift + cap:] == b"\xa5" * (len(host) - shift - cap)


def stream_of(keys, counts, k):
    """oracle_stream for many pairs: counter bytes and key bytes placed by offset."""
    kb, W = (k + 3) // 4, keys.shape[1]
    x = keys.copy()
    x[:, -1] <<= np.uint64(2 * (32 * W - k))
    body = x.astype(">u8").view(np.uint8).reshape(-1, 8 * W)[:, :kb]
    big = counts >= 255
    size = 1 + kb + 4 * big.astype(np.int64)
    at = np.cumsum(size) - size
    out = np.zeros(int(size.sum()), dtype=np.uint8)
    out[at] = np.where(big, 255, counts).astype(np.uint8)
    head = counts.astype(">u4").view(np.uint8).reshape(-1, 4)
    for j in range(4):
        out[at[big] + 1 + j] = head[big, j]
    for j in range(kb):
        out[at + size - kb + j] = body[:, j]
    return out.tobytes()


@pytest.mark.parametrize("k", [3, 28, 32, 33, 61, 64, 65])
def test_large_tiles(k):
    """From 2 M pairs on a tile takes several rounds, of two pairs a thread up to k = 64."""
    rng = np.random.default_rng(k)
    few = random_pairs(rng, 500, k)
    assert stream_of(*few, k) == oracle_stream(*few, k)
    n = 256 * 8192 + 1024 * 9 + 77
    keys, counts = random_pairs(rng, n, k)
    kd, cd = device_pairs(keys, counts)
    assert g.records(kd, cd, n, k).cpu().numpy().tobytes() == stream_of(keys, counts, k)
