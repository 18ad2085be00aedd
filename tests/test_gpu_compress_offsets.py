"""Fields whose values lie far from 0: the first cell of every chunk then has a
code past the packed arithmetic's limits, or an escape, while the rest of its
layer does not.  Streams are compared with the oracle's, byte for byte.

With eb = 0.5 the integers are the (integer) values themselves.
"""
import numpy as np
import pytest
import torch

import paper_2304_12557_amd as fz
from oracle import oracle as O

pytestmark = pytest.mark.gpu

SHAPES = [(33, 37, 70), (2, 1, 3), (75, 1030), (1, 2050), (70_001,), (1,)]
# around a code's 32767, the packed limits of 3-D and 2-D, and the rounding's 2^22
OFFSETS = [8191, 8192, 16384, 32767, 32768, -32767, -32768, 100_000, -100_000, 4_194_000, 4_194_304]


def field(shape, off, kind):
    rng = np.random.default_rng(abs(off) + len(shape))
    x = rng.integers(-20, 21, shape) + off
    if kind == "spikes":  # escapes of other cells of the first layer, and of later ones
        x.reshape(-1)[rng.integers(0, x.size, 3)] += 300_000
    elif kind == "steep":  # the first step itself leaves the packed arithmetic
        x += (np.arange(shape[-1]) * 997).astype(x.dtype)
    return x.astype(np.float64)


def same(buf, ref, st, what):
    info = fz.stream_info(buf)
    assert info["status"] == st, what
    if st == 0:
        s = buf[:fz.stream_size(buf)].cpu().numpy()
        assert s.size == ref.size and np.array_equal(s, ref), what


@pytest.mark.parametrize("kind", ["flat", "spikes", "steep"])
@pytest.mark.parametrize("shape", SHAPES)
def test_offsets(shape, kind):
    xs = [field(shape, off, kind) for off in OFFSETS]
    fs = [torch.from_numpy(x.astype(np.float32)).cuda() for x in xs]
    b = fz.Batch.compress([(f, 0.5, "abs", None) for f in fs])
    outs = b.run()
    for off, x, f, out in zip(OFFSETS, xs, fs, outs):
        print("case", shape, kind, off, flush=True)
        ref, st = O.compress(f.cpu().numpy(), 0.5, O.EB_ABS)
        same(fz.compress(f, 0.5, "abs"), ref, st, off)
        same(out, ref, st, ("batch", off))
        for g in (False, True):
            ref, st = O.compress(f.cpu().numpy(), 0.5, O.EB_ABS, global_lorenzo=g)
            same(fz.compress(f, 0.5, "abs", global_lorenzo=g), ref, st, (off, g))
        ref, st = O.compress_f64(x, 0.5, O.EB_ABS)
        same(fz.compress(torch.from_numpy(x).cuda(), 0.5, "abs"), ref, st, ("double", off))
        pw = f.abs() + 1
        ref, st = O.compress(pw.cpu().numpy(), 1e-3, O.EB_PWREL)
        same(fz.compress(pw, 1e-3, "pwrel"), ref, st, ("pwrel", off))
    b.close()


@pytest.mark.parametrize("others", [1022, 1023, 1024])
def test_first_cell_and_the_cap(others):
    x = np.full(32768, 50_000.0, dtype=np.float32)  # the first cell is an escape
    x[20_000:20_000 + others] += 40_000 * (np.arange(others) % 2 == 0)  # `others` + (odd) jumps of 40000
    ref, st = O.compress(x, 0.5, O.EB_ABS)
    same(fz.compress(torch.from_numpy(x).cuda(), 0.5, "abs"), ref, st, others)
