"""The decompressor's workgroups (a chunk's steps shared out over 8 or 16
waves): stores at the edges of its tiles into outputs of any alignment, and
streams whose escape pairs or chunk table do not fit.

A field of at most 256 chunks takes the 16-wave form, a larger one the 8-wave
form.  Expected values come from the oracle (fp32, bit for bit) or, for fp64,
from the decompression of the same stream into an aligned output.
"""
import numpy as np
import pytest
import torch

import paper_2304_12557_amd as fz
from oracle import oracle as O
import synth

pytestmark = pytest.mark.gpu


def offset_view(shape, dtype, off):
    """A contiguous tensor of `shape` that starts `off` values into guarded
    memory, and the guard around it."""
    n = int(np.prod(shape))
    big = torch.full((n + off + 64,), -7.0, dtype=dtype, device="cuda")
    return big[off:off + n].view(shape), big


# row lengths around a tile's 64 (3-D), 1024 (2-D) and 2048 (1-D) values and
# around whole 16-byte pieces; steps cut by the field's edge
SHAPES = [(17, 33, 63), (16, 32, 64), (5, 40, 65), (16, 31, 130), (3, 4, 1), (33, 1023), (32, 1024), (31, 1025), (1, 2),
          (2, 4097), (1,), (2047,), (2049,), (32768,), (70_003,)]
BIG = [(100, 300, 301), (266, 33_001), (8_500_001,)]  # 3-D 350, 2-D 297, 1-D 260 chunks


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("shape", SHAPES + BIG)
def test_any_output_alignment(shape, off):
    x = synth.sine_field(shape, seed=11 + len(shape))
    print("case", shape, off, flush=True)
    xt = torch.from_numpy(x).cuda()
    s = fz.compress(xt, 1e-3, "rel")
    ref, st = O.compress(x, 1e-3, O.EB_REL, threads=8)
    assert st == 0
    yo, e = O.decompress(ref, shape, threads=8)
    assert e == 0
    y, big = offset_view(shape, torch.float32, off)
    err = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    fz.decompress(s, shape, out=y, err=err)
    assert int(err.item()) == 0
    assert np.array_equal(y.cpu().numpy().view(np.uint32), yo.view(np.uint32))
    g = big.cpu().numpy()
    assert (g[:off] == -7).all() and (g[off + x.size:] == -7).all()
    s64 = fz.compress(xt.double(), 1e-3, "rel")
    want = fz.decompress(s64, shape, dtype=torch.float64)
    y, big = offset_view(shape, torch.float64, off)
    fz.decompress(s64, shape, out=y)
    assert torch.equal(y, want)
    assert float((y - xt.double()).abs().max()) <= 1.001e-3 * float(x.max() - x.min() if x.size > 1 else abs(x).max())
    g = big.cpu().numpy()
    assert (g[:off] == -7).all() and (g[off + x.size:] == -7).all()


def spikes(chunks):
    """A 1-D field of whole chunks and 100 values whose second chunk and last
    chunk hold escapes in several steps."""
    shape = (32768 * chunks + 100,)
    x = np.zeros(shape, dtype=np.float32)
    x[32768 + 40:2 * 32768:1500] = 100000.0  # two escapes each, in many steps
    x[-60] = 100000.0
    return x


def pairs_of(s, shape, c):
    """Byte offset of chunk c's pairs in stream s, and their number."""
    n_chunks = -(-shape[0] // 32768)
    off, nout = np.frombuffer(s[128 + 8 * c:128 + 8 * c + 8].tobytes(), np.uint32)
    flags = 128 + (8 * n_chunks + 15) // 16 * 16 + 512 * c
    nnz = int(np.unpackbits(s[flags:flags + 512]).sum())
    return fz.header_bytes(shape) + 16 * (int(off) + nnz), int(nout)


def swap(p):
    p[[4, 6]] = p[[6, 4]]
    p[[5, 7]] = p[[7, 5]]


def move(p):
    p[4] += 2  # a cell whose code is no escape


def repeat(p):
    p[6] = p[4]


def past(p):
    p[-2] = 40000  # no such code


def earlier(p):
    p[-2] = 41  # the last pair claims a cell of the first step


@pytest.mark.parametrize("chunks", [3, 300])
@pytest.mark.parametrize("spoil", [swap, move, repeat, past, earlier])
def test_escape_pairs_that_do_not_match(chunks, spoil):
    x = spikes(chunks)
    buf = fz.compress(torch.from_numpy(x).cuda(), 0.5, "abs")
    s = buf[:fz.stream_size(buf)].cpu().numpy()
    y = fz.decompress(torch.from_numpy(s).cuda(), x.shape).cpu().numpy()
    assert np.abs(y - x).max() <= 0.5
    at, nout = pairs_of(s, x.shape, 1)
    assert nout > 20
    p = s[at:at + 8 * nout].view(np.uint32)
    spoil(p)
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.full(x.shape, -7.0, device="cuda")
    fz.decompress(torch.from_numpy(s).cuda(), x.shape, out=out, err=err)
    assert int(err.item()) == 6
    out = out.cpu().numpy()
    assert (out[32768:2 * 32768] == -7).all()  # the bad chunk is not written
    assert np.array_equal(out[:32768], y[:32768]) and np.array_equal(out[2 * 32768:], y[2 * 32768:])


@pytest.mark.parametrize("chunks", [5, 300])
def test_shifted_table_stays_inside_the_payload(chunks):
    """Chunk offsets that follow from one another but lie past the payload:
    every chunk from there on is refused, not only those at the shift's ends."""
    x = spikes(chunks)
    buf = fz.compress(torch.from_numpy(x).cuda(), 0.5, "abs")
    s = buf[:fz.stream_size(buf)].cpu().numpy()
    n_chunks = chunks + 1
    tab = s[128:128 + 8 * n_chunks].view(np.uint32)
    tab[2 * 2::2] += 1 << 20
    err = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.full(x.shape, -7.0, device="cuda")
    fz.decompress(torch.from_numpy(s).cuda(), x.shape, out=out, err=err)
    assert int(err.item()) == 6
    out = out.cpu().numpy()
    assert (out[32768:] == -7).all()
    assert (out[:32768] == 0).all()
