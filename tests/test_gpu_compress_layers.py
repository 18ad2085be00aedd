"""The compressor's layers: differences at and past the limits of the packed
16-bit arithmetic, integers past the biased rounding's range, chunks whose
payload does not fit the staging buffer, and escapes on each of these ways.

With eb = 0.5 the integers are the (integer) values themselves.  Streams are
compared with the oracle's, byte for byte, field by field and in one batch.
"""
import numpy as np
import pytest
import torch

import paper_2304_12557_amd as fz
from oracle import oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [(33, 37, 70), (16, 32, 64), (75, 1030), (70_001,)]
REACH = {3: 4, 2: 2, 1: 1}  # how often a difference along the sweep counts in a checkerboard's delta


def checker(shape, first, amp, offset):
    """Zeros, and from index `first` of the sweep dimension on a checkerboard
    of +-amp in the other dimensions; all moved by `offset`."""
    x = np.zeros(shape, dtype=np.float32)
    sign = np.indices(shape[1:]).sum(axis=0) % 2 * 2 - 1 if len(shape) > 1 else 1
    x[first:] = amp * sign
    return x + np.float32(offset)


def noise(shape, span, offset, seed=3):
    return (np.random.default_rng(seed).integers(-span, span + 1, shape) + offset).astype(np.float32)


def fields(shape):
    reach = REACH[len(shape)]
    lim = 32767 // reach
    out = [checker(shape, first, amp, off)
           for first in sorted({0, 1, 3, 4, 6, 7, 15}) if first < shape[0]
           for amp in (lim, lim + 1) for off in (0, 5_000_000)]
    # codes of all 16 bits without an escape, with some, and beyond the cap
    span = 32767 >> len(shape)
    out += [noise(shape, s, off) for s in (span, span + span // 8, 4 * span) for off in (0, 5_000_000)]
    # one layer in 32 bits between packed ones
    x = noise(shape, 20, 0)
    x.reshape(-1)[x.size // 2] = 40_000
    return out + [x]


def stream(buf):
    info = fz.stream_info(buf)
    return info["status"], buf[:fz.stream_size(buf)].cpu().numpy() if info["status"] == 0 else None


def check(buf, x, what):
    ref, st = O.compress(x, 0.5, O.EB_ABS, threads=8)
    got, s = stream(buf)
    assert got == st, what
    if st == 0:
        assert s.size == ref.size and np.array_equal(s, ref), what


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("shape", SHAPES)
def test_layers_against_the_oracle(shape, off):
    for i, x in enumerate(fields(shape)):
        print("case", shape, off, i, flush=True)
        big = torch.zeros(x.size + 8, device="cuda")
        xt = big[off:off + x.size].view(shape)
        xt.copy_(torch.from_numpy(x))
        check(fz.compress(xt, 0.5, "abs"), x, i)


def test_layers_in_one_batch():
    xs = [x for shape in SHAPES for x in fields(shape)]
    print("batch of", len(xs), flush=True)
    b = fz.Batch.compress([(torch.from_numpy(x).cuda(), 0.5, "abs", None) for x in xs])
    for i, (buf, x) in enumerate(zip(b.run(), xs)):
        check(buf, x, i)
    b.close()
