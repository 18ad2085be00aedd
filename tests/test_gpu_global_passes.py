"""The passes around the chunk kernels of the field-global predictor: runs and
faces at every edge of a chunk, inputs and outputs of any alignment, lines of
more segments than one pass of the carries takes, and bad values seen only as
some chunk's face.  Expected values come from the oracle, bit for bit.
"""
import numpy as np
import pytest
import torch

import paper_2304_12557_amd as fz
from oracle import oracle as O
import synth

pytestmark = pytest.mark.gpu

MODES = {"abs": O.EB_ABS, "rel": O.EB_REL, "pwrel": O.EB_PWREL}
# extents around a run's 4 values, a wave's rows, planes and columns and a chunk's box
SHAPES = [(17, 33, 65), (16, 36, 66), (33, 31, 67), (5, 64, 3), (65, 1, 260), (33, 1025), (40, 1283), (64, 2048), (9, 253),
          (32769,), (65_536 + 2047,), (32768 * 2 + 3,)]
# carries: 300 segments of one line; 94 of many and of few lines; 44 along the slowest axis; 17 rows of 64
LONG = [(9_830_007,), (3000, 1100), (3000, 5), (700, 3, 70), (3, 700, 131), (2, 2, 1200)]


def view(shape, off):
    n = int(np.prod(shape))
    big = torch.full((n + off + 64,), -7.0, device="cuda")
    return big[off:off + n].view(shape), big


@pytest.mark.parametrize("off,mode,eb", [(0, "rel", 1e-3), (1, "abs", 1e-3), (3, "pwrel", 1e-2)])
@pytest.mark.parametrize("shape", SHAPES + LONG)
def test_any_edge_and_alignment(shape, off, mode, eb):
    print("case", shape, off, mode, flush=True)
    x = synth.sine_field(shape, seed=len(shape) + off) + np.float32(0.25)
    ref, st = O.compress(x, eb, MODES[mode], threads=8, global_lorenzo=True)
    assert st == 0
    xt, _ = view(shape, off)
    xt.copy_(torch.from_numpy(x))
    s = fz.compress(xt, eb, mode, global_lorenzo=True)
    got = s[:fz.stream_size(s)].cpu().numpy()
    assert got.size == ref.size and np.array_equal(got, ref)
    yo, e = O.decompress(ref, shape, threads=8)
    assert e == 0
    y, big = view(shape, off)
    fz.decompress(s, shape, out=y, global_lorenzo=True)
    assert np.array_equal(y.cpu().numpy().view(np.uint32), yo.view(np.uint32))
    g = big.cpu().numpy()
    assert (g[:off] == -7).all() and (g[off + x.size:] == -7).all()


@pytest.mark.parametrize("at", [(0, 0, 0), (15, 31, 63), (16, 31, 64), (39, 69, 129), (15, 40, 0)])
@pytest.mark.parametrize("bad,status", [(np.nan, O.ERR_NONFINITE), (-np.inf, O.ERR_NONFINITE), (1e15, O.ERR_EB_RANGE)])
def test_bad_value_anywhere(at, bad, status):
    x = synth.sine_field((40, 70, 130), seed=5)
    x[at] = bad
    print("case", at, bad, flush=True)
    _, st = O.compress(x, 1e-3, O.EB_ABS, global_lorenzo=True)
    s = fz.compress(torch.from_numpy(x).cuda(), 1e-3, "abs", global_lorenzo=True)
    assert fz.stream_info(s)["status"] == st == status
