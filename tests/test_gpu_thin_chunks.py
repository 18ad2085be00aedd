"""Decompression of fields whose last layer of chunks is thin: as many waves as it
has pairs of steps run one of its chunks, and a workgroup several chunks.

More than 256 chunks each (fewer take 16 waves whatever their depth); escapes in
the first and the last step; the oracle's values bit for bit.
"""
import numpy as np
import pytest
import torch

import paper_2304_12557_amd as fz
from oracle import oracle as O
import synth

pytestmark = pytest.mark.gpu

SHAPES = [(n, 1030, 530) for n in (1, 2, 3, 4, 5, 8, 9, 14, 15, 16, 17)] + [(n, 300_001) for n in (1, 2, 4, 5, 8, 13, 28, 29, 32, 33)]
# a thin layer of more chunks than are at work at once, and whole layers before
# one that does not fit the last round behind them; the last workgroup not full
SHAPES += [(n, 1030, 1060) for n in (1, 2, 3, 5, 8)] + [(n, 560_001) for n in (1, 3, 8, 15)]
SHAPES += [(n, 530, 1030) for n in (18, 20, 21, 24, 25, 33)] + [(n, 290_001) for n in (34, 37, 40, 47, 49, 65)]
ALIGNED = [(33, 530, 1024), (36, 512, 1024), (38, 290 * 1024), (2, 1056, 576), (6, 1056, 576), (3, 264 * 1024), (12, 264 * 1024)]  # rows of whole lines: streaming stores


def field(shape, escapes):
    x = np.round(synth.sine_field(shape, seed=sum(shape)) * 200).astype(np.float32)
    if escapes:
        flat = x.reshape(-1)
        flat[1000::50_021] += 70_000
        x[0, ..., -1] += 50_000
        x[-1, ..., 3] -= 60_000
    return x


@pytest.mark.parametrize("escapes", [False, True])
@pytest.mark.parametrize("shape", SHAPES + ALIGNED)
def test_thin_fields(shape, escapes):
    x = field(shape, escapes)
    print("case", shape, escapes, flush=True)
    ref, st = O.compress(x, 0.5, O.EB_ABS, threads=8)
    assert st == 0
    s = torch.from_numpy(ref).cuda()
    guard = torch.full((x.size + 128,), -7.0, device="cuda")
    y = guard[64:64 + x.size].view(shape)
    err = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    fz.decompress(s, shape, out=y, err=err)
    assert int(err.item()) == 0
    assert np.array_equal(y.cpu().numpy(), x)
    assert bool((guard[:64] == -7).all()) and bool((guard[64 + x.size:] == -7).all())


BAD = [(2, 1030, 530), (7, 1030, 530), (3, 300_001), (2, 1030, 1060), (4, 1030, 1060), (7, 1030, 1060), (3, 560_001), (15, 560_001)]


@pytest.mark.parametrize("shape", BAD)
def test_a_pair_that_does_not_match(shape):
    x = field(shape, True)
    ref, st = O.compress(x, 0.5, O.EB_ABS, threads=8)
    assert st == 0
    tab = ref[128:].view(np.uint8)[:8].view(np.uint32)
    nout = int(tab[1])
    assert nout > 0 and int(tab[0]) == 0
    n_chunks = fz.stream_info(ref[:128].tobytes())["n_chunks"]
    flags = 128 + (8 * n_chunks + 15) // 16 * 16
    nnz = int(np.unpackbits(ref[flags:flags + 512]).sum())
    pairs = ref[fz.header_bytes(shape) + 16 * nnz:][:8 * nout].view(np.uint32)
    pairs[-2] = 16 * 2048 - 1  # a cell of a step the field does not reach
    y = torch.full(shape, -7.0, device="cuda")
    err = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    fz.decompress(torch.from_numpy(ref).cuda(), shape, out=y, err=err)
    assert int(err.item()) == 6
    box = (32, 64) if len(shape) == 3 else (1024,)
    first = tuple([slice(None)] + [slice(0, b) for b in box])
    got = y.cpu().numpy()
    assert (got[first] == -7).all()  # the bad chunk is not written
    got[first] = x[first]
    assert np.array_equal(got, x)


@pytest.mark.parametrize("chunk", [0, 1, 6])
@pytest.mark.parametrize("shape", BAD)
def test_a_flag_past_the_field(shape, chunk):
    """One chunk of a workgroup is refused before its first barrier, the others
    go on."""
    x = field(shape, True)
    ref, st = O.compress(x, 0.5, O.EB_ABS, threads=8)
    assert st == 0
    n_chunks = fz.stream_info(ref[:128].tobytes())["n_chunks"]
    flags = 128 + (8 * n_chunks + 15) // 16 * 16 + 512 * chunk
    ref[flags + 511] ^= 0x80  # a brick of the last layer, which the field does not reach
    y = torch.full(shape, -7.0, device="cuda")
    err = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    print("case", shape, chunk, flush=True)
    fz.decompress(torch.from_numpy(ref).cuda(), shape, out=y, err=err)
    assert int(err.item()) == 6
    box = (32, 64) if len(shape) == 3 else (1024,)
    per_row = -(-shape[-1] // box[-1])
    org = (32 * (chunk // per_row), 64 * (chunk % per_row)) if len(shape) == 3 else (1024 * chunk,)
    bad = tuple([slice(None)] + [slice(o, o + b) for o, b in zip(org, box)])
    got = y.cpu().numpy()
    assert (got[bad] == -7).all()
    got[bad] = x[bad]
    assert np.array_equal(got, x)
