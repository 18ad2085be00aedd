"""The exact values at which the compressor's packed path, escape cap and forms
change, byte for byte against the oracle (eb = 0.5: the integers are the values).

* Steps whose differences along the sweep pass the packed limit (8191 in 3-D,
  16383 in 2-D) are looked at in 256ths: deltas around 126 * 256 (the last one
  that passes there) and 32767 (the last that is no escape), and differences
  along the sweep around 2^20, where the 256ths no longer fit.
* A chunk of 1023, 1024 and 1025 escapes, its first cell among them.
* Fields of 256 and 257 chunks (16 and 8 waves a chunk in decompression).
"""
import numpy as np
import pytest
import torch

import paper_2304_12557_amd as fz
from oracle import oracle as O

pytestmark = pytest.mark.gpu

DELTAS = [s * d for d in (32255, 32256, 32257, 32511, 32512, 32513, 32766, 32767, 32768, 32769) for s in (1, -1)]


def same(buf, ref, st, what):
    info = fz.stream_info(buf)
    assert info["status"] == st, (what, info["status"], st)
    if st == 0:
        s = buf[:fz.stream_size(buf)].cpu().numpy()
        assert s.size == ref.size and np.array_equal(s, ref), what


def check(x, what, n_escapes=None):
    print("case", what, flush=True)
    x32 = x.astype(np.float32)
    assert np.array_equal(x32, x)
    ref, st = O.compress(x32, 0.5, O.EB_ABS)
    if n_escapes is not None and st == 0:
        assert fz.stream_info(ref[:128].tobytes())["n_outliers"] == n_escapes, what
    same(fz.compress(torch.from_numpy(x32).cuda(), 0.5, "abs"), ref, st, what)
    b = fz.Batch.compress([(torch.from_numpy(x32).cuda(), 0.5, "abs", None)])
    same(b.run()[0], ref, st, (what, "batch"))
    b.close()
    ref, st = O.compress_f64(x.astype(np.float64), 0.5, O.EB_ABS)
    same(fz.compress(torch.from_numpy(x.astype(np.float64)).cuda(), 0.5, "abs"), ref, st, (what, "double"))


# one chunk; cut by the field's edge; several
SHAPES = [(16, 32, 64), (9, 30, 61), (17, 33, 65), (32, 1024), (21, 1000), (33, 1025)]


@pytest.mark.parametrize("at", [0, 2, 5])  # the step that jumps: the first, in layer 0, in layer 1
@pytest.mark.parametrize("shape", SHAPES)
def test_deltas_past_the_packed_limit(shape, at):
    rank = len(shape)
    row = at if rank == 3 else 2 * at
    jump = 9000 if rank == 3 else 17_000
    xs = []
    for d in DELTAS:
        x = np.zeros(shape, dtype=np.int64)
        x[row:] += jump                    # the sweep difference of a whole step
        cell = (3, 13) if rank == 3 else (77,)
        x[(row,) + cell] += d              # the delta there d, its neighbours' -d or d
        x[(slice(row + 1, None),) + cell] += d
        xs.append(x)
    for d, x in zip(DELTAS, xs):
        check(x, (shape, at, d))


@pytest.mark.parametrize("at", [0, 2, 5])
@pytest.mark.parametrize("shape", SHAPES)
def test_sweep_differences_around_2_20(shape, at):
    rank = len(shape)
    row = at if rank == 3 else 2 * at
    for top in (2 ** 20 - 1, 2 ** 20, 2 ** 20 + 1, -2 ** 20 - 1, -2 ** 20, -2 ** 20 + 1):
        x = np.zeros(shape, dtype=np.int64)
        box = (min(32, shape[1]), min(64, shape[2])) if rank == 3 else (min(1024, shape[1]),)
        g = abs(top) // (sum(box) - len(box))  # a ramp from 0 to about `top` over the chunk's step
        ramp = g * np.indices(shape[1:]).sum(axis=0) * (1 if top > 0 else -1)
        last = tuple(b - 1 for b in box)
        assert abs(ramp[last]) <= abs(top) and g < 32000
        ramp[last] = top
        x[row:] += ramp
        check(x, (shape, at, top))


@pytest.mark.parametrize("start", [9, 20_000, 31_744])
@pytest.mark.parametrize("jumps", [1022, 1023, 1024])
def test_exact_escape_counts(start, jumps):
    """The first cell and `jumps` jumps of 40000, the last run up to the end."""
    jumps = min(jumps, 32768 - start)
    x = np.full(32768, 50_000, dtype=np.int64)
    x[start:] += 40_000 * (np.minimum(np.arange(32768 - start), jumps - 1) % 2 == 0)
    total = 1 + int((np.abs(np.diff(x)) > 32767).sum())
    assert total == 1 + jumps
    check(x, (start, total), total)
    x32 = x.astype(np.float32)
    ref, st = O.compress(x32, 0.5, O.EB_ABS)
    assert (st == 0) == (total <= 1024)
    if st == 0:
        err = torch.full((1,), 5, dtype=torch.int32, device="cuda")
        y = fz.decompress(torch.from_numpy(ref).cuda(), x.shape, err=err)
        assert int(err.item()) == 0 and np.array_equal(y.cpu().numpy(), x32)


@pytest.mark.parametrize("shape", [(256 * 32768,), (256 * 32768 + 1,), (32, 256 * 1024), (32 * 257, 1000), (16, 32, 64 * 256),
                                   (16 * 257, 30, 61)])
def test_256_and_257_chunks(shape):
    rng = np.random.default_rng(len(shape))
    x = rng.integers(-40, 41, shape).astype(np.float32)
    x.reshape(-1)[::70_001] += 60_000
    print("case", shape, flush=True)
    ref, st = O.compress(x, 0.5, O.EB_ABS, threads=8)
    assert st == 0 and fz.stream_info(ref[:128].tobytes())["n_chunks"] in (256, 257)
    same(fz.compress(torch.from_numpy(x).cuda(), 0.5, "abs"), ref, st, shape)
    err = torch.full((1,), 5, dtype=torch.int32, device="cuda")
    y = fz.decompress(torch.from_numpy(ref).cuda(), shape, err=err)
    assert int(err.item()) == 0 and np.array_equal(y.cpu().numpy(), x)
