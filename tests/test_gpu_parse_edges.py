"""The copy and newline kernels of the parser on lines of every short length:
16-byte output chunks that hold parts of one, two, three and more lines, empty
lines between them, newlines at both ends of a lane's and a wave's bytes, and
texts that start and end inside a 16-byte word. Bytes equal the oracle's."""
import numpy as np
import pytest

from paper_1607_06618_amd import gerbil as g
from test_gpu_parse import compare

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    g.load()


def line(rng, n):
    return rng.choice(np.frombuffer(b"ACGTN", dtype=np.uint8), n).tobytes()


@pytest.mark.parametrize("shift", [0, 1, 15])
@pytest.mark.parametrize("longest", [3, 9, 17, 40, 150])
@pytest.mark.parametrize("end", [b"\n", b"\r\n"])
def test_fasta_line_lengths(longest, end, shift):
    rng = np.random.default_rng(longest)
    out = []
    for i in range(6000):
        if i % 7 == 0:
            out.append(b">r%d" % i if rng.random() < 0.5 else b">")
        out.append(line(rng, int(rng.integers(0, longest + 1))))
    compare(end.join(out), shift=shift)


@pytest.mark.parametrize("shift", [0, 7])
@pytest.mark.parametrize("longest", [1, 15, 16, 33, 300])
def test_fastq_read_lengths(longest, shift):
    rng = np.random.default_rng(longest)
    out = []
    for i in range(3000):
        s = line(rng, int(rng.integers(0 if longest > 1 else 1, longest + 1)))
        out += [b"@" + b"x" * int(rng.integers(0, 20)), s, b"+", b"I" * len(s)]
    compare(b"\n".join(out) + b"\n", shift=shift)


@pytest.mark.parametrize("gap", [15, 16, 17, 1023, 1024, 1025, 4095, 4096])
def test_newlines_at_lane_and_wave_edges(gap):
    compare(b">a\n" + b"\n".join(b"A" * gap for _ in range(100)) + b"\n>b\nC")


@pytest.mark.parametrize("lines", [1, 3, 300, 2100])
def test_long_lines_are_shared_out(lines):
    """Lines of more than a slice of a copy tile, among empty and short ones."""
    rng = np.random.default_rng(lines)
    out = []
    for i in range(lines):
        out += [b">", b"", line(rng, 3_000_000 // lines + int(rng.integers(0, 40))), b"AC"]
    compare(b"\n".join(out))


@pytest.mark.parametrize("fmt", [g.GERBIL_FORMAT_DETECT, g.GERBIL_FORMAT_FASTQ, g.GERBIL_FORMAT_FASTA])
@pytest.mark.parametrize("text", [b"", b"\n", b">", b"@\n\n+\n\n"])
def test_first_offset_is_written(text, fmt):
    """Offsets [0, n_reads] are the call's, whatever the buffer held: an empty text has the one offset 0."""
    import ctypes

    import torch
    n = len(text)
    t = torch.zeros(64, dtype=torch.uint8, device="cuda")
    if n:
        t[:n] = torch.frombuffer(bytearray(text), dtype=torch.uint8).cuda()
    info_d = torch.zeros(ctypes.sizeof(g.gerbil_parsed), dtype=torch.uint8, device="cuda")
    ws = torch.empty(max(256, g.gerbil_parse_workspace(n, n + 1)), dtype=torch.uint8, device="cuda")
    seq = torch.empty(n + 1, dtype=torch.uint8, device="cuda")
    offsets = torch.full((n + 2,), 77, dtype=torch.int64, device="cuda")
    assert g.gerbil_parse(t.data_ptr(), n, fmt, ws.data_ptr(), ws.numel(), n + 1, seq.data_ptr(), n, offsets.data_ptr(),
                          n + 1, info_d.data_ptr(), g._stream_handle(None)) == g.GERBIL_OK
    info = g.gerbil_parsed.from_buffer_copy(info_d.cpu().numpy().tobytes())
    if info.status == 0:
        assert int(offsets[0]) == 0 and int(offsets[info.n_reads]) == info.n_bytes
