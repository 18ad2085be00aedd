"""Extents each inside their own limit whose chunk counts multiply past 64 bits
are refused like any field of 2^31 chunks or more (CPU only)."""
import ctypes

import pytest

import paper_2304_12557_amd as fz

P = 4096  # a pointer that no call gets to use


@pytest.mark.parametrize("n", [
    (1 << 40, 1 << 40, 1 << 24),           # 2^89 chunks: 0 modulo 2^64
    (1 << 40, 1 << 40, 1),                 # 2^71 chunks
    (1 << 40, 1 << 40, (1 << 25) - 1),
    (1 << 39, 1 << 33, 1 << 24),
    (16 * 4295098370, 32 * 4294836226, 64),  # 2^64 + 4 chunks
    (16 * 641, 32 * 6700417 * 64, 64),     # (2^32 + 1) * 64 chunks
])
def test_chunk_counts_past_64_bits(n):
    L = fz.lib()
    d = fz.FzDims(3, 0, (ctypes.c_uint64 * 3)(*n))
    assert L.fz_compress_bound(ctypes.byref(d)) == 0
    assert L.fz_header_bytes(ctypes.byref(d)) == 0
    assert L.fz_stream_bound(ctypes.byref(d)) == 0
    assert L.fz_compress(P, ctypes.byref(d), 1e-3, 1, P, None) == 1
    assert L.fz_decompress(P, 1 << 40, P, ctypes.byref(d), None, None) == 1


def test_the_largest_fields_stay_accepted():
    L = fz.lib()
    for n in ((1 << 35, 1, 1), ((16 << 31) - 16, 1, 1), (1, (32 << 31) - 32, 1)):  # up to 2^31 - 1 chunks
        d = fz.FzDims(3, 0, (ctypes.c_uint64 * 3)(*n))
        chunks = -(-n[0] // 16) * -(-n[1] // 32)
        assert (L.fz_compress_bound(ctypes.byref(d)) > 0) == (chunks < 1 << 31), n
