"""Decompression of fields whose chunks do not fit one launch (its threads are
counted in 32 bits): a column of 2^27 + 16 cells is 2^23 + 1 chunks.

The stream is put together from the oracle's stream of the last chunk: all
others hold zeros, which take no payload.  The runtime does not refuse a launch
past that limit: it runs what is left modulo 2^32 threads, here one workgroup.
"""
import struct

import numpy as np
import pytest
import torch

import paper_2304_12557_amd as fz
from oracle import oracle as O

pytestmark = pytest.mark.gpu

CHUNKS = (1 << 23) + 1
SHAPE = (16 * CHUNKS, 1, 1)
LAST = np.array([5, 4, -3, 0, 7, 7, 100, 2, -2, 1, 0, 0, 3, 3, 3, -40], dtype=np.float32).reshape(16, 1, 1)


def stream(dtype, glob):
    """Device stream of SHAPE: LAST (eb 0.5 ABS: its own integers) behind zeros."""
    if dtype == torch.float64:
        one, st = O.compress_f64(LAST.astype(np.float64), 0.5, O.EB_ABS)
    else:
        one, st = O.compress(LAST, 0.5, O.EB_ABS, global_lorenzo=glob)
    assert st == 0
    head, flags, payload = one[:128].copy(), one[144:144 + 512], one[144 + 512:]
    payload_off = fz.header_bytes(SHAPE)
    head[16:40] = np.frombuffer(struct.pack("<3Q", *SHAPE), dtype=np.uint8)
    head[72:76] = np.frombuffer(struct.pack("<I", CHUNKS), dtype=np.uint8)
    head[96:104] = np.frombuffer(struct.pack("<Q", payload_off + payload.size), dtype=np.uint8)
    s = torch.zeros(payload_off + payload.size, dtype=torch.uint8, device="cuda")
    s[:128] = torch.from_numpy(head).cuda()
    s[payload_off - 512:payload_off] = torch.from_numpy(flags.copy()).cuda()
    s[payload_off:] = torch.from_numpy(payload.copy()).cuda()
    return s


def check(y, err=None):
    torch.cuda.synchronize()
    assert err is None or int(err.item()) == 0
    assert np.array_equal(y[-16:].cpu().numpy().astype(np.float32), LAST)
    assert int(torch.count_nonzero(y[:-16])) == 0


@pytest.mark.parametrize("dtype,glob", [(torch.float32, False), (torch.float64, False), (torch.float32, True)])
def test_fields(dtype, glob):
    s = stream(dtype, glob)
    print("case", dtype, glob, flush=True)
    y = torch.full(SHAPE, 9.0, dtype=dtype, device="cuda")
    err = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    fz.decompress(s, SHAPE, out=y, err=err, dtype=dtype, global_lorenzo=glob)
    check(y, err)


def test_batch():
    s = stream(torch.float32, False)
    y = torch.full(SHAPE, 9.0, dtype=torch.float32, device="cuda")
    small = np.arange(40, dtype=np.float32).reshape(5, 8)
    t, st = O.compress(small, 0.5, O.EB_ABS)
    z = torch.zeros((5, 8), dtype=torch.float32, device="cuda")
    ts = torch.from_numpy(t).cuda()
    err = torch.full((1,), 77, dtype=torch.int32, device="cuda")
    b = fz.Batch.decompress([(s, SHAPE, y, err), (ts, (5, 8), z, None)])
    b.run()
    check(y, err)
    assert np.array_equal(z.cpu().numpy(), small)
    b.close()
