"""Occupancy and spills the present kernels are built around (CPU only), from the
compiler's report that build() leaves beside the library.

* A decompression workgroup of 8 waves shares its CU with another one: 4 waves
  per SIMD, so at most 128 registers a lane, and at most half of a CU's 160 KB of
  LDS.  The 16-wave form has a CU to itself.
* The field-global passes run workgroups of 16 waves: at least 4 per SIMD.
* The compression kernels that are launched (16-byte loads) hold a layer's planes
  in registers at 2 waves per SIMD.  A few values spill around their out-of-line
  calls; the ceilings keep that from growing into the loop (two more in one kernel
  cost 2 % of 100x500x500).
"""
import json
import os

import pytest

PATH = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_12557_amd",
                    "kernel_resources.json")
KB = 1024


@pytest.fixture(scope="module")
def res():
    if not os.path.exists(PATH):
        pytest.skip("no kernel resource report: run build() first")
    with open(PATH) as fh:
        return json.load(fh)


def family(res, name):
    out = {k: v for k, v in res.items() if k.startswith("_ZN2fz%d%s" % (len(name), name))}  # (the length ends the name)
    assert out, name
    return out


@pytest.mark.parametrize("name,lds", [("k_decompress", 80 * KB), ("k_decompress_ahead", 80 * KB), ("k_decompress64", 80 * KB),
                                      ("k_decompress_int", 80 * KB), ("k_batch_decompress", 80 * KB), ("k_decompress_split", 160 * KB)])
def test_decompression(res, name, lds):
    for k, v in family(res, name).items():
        assert v["waves_per_simd"] >= 4 and v["vgprs"] <= 128, (k, v)
        assert v["lds_bytes"] <= lds, (k, v)
        assert v["vgpr_spills"] == 0 and v["scratch_bytes_per_lane"] == 0, (k, v)


@pytest.mark.parametrize("name", ["k_face", "k_seg_final", "k_seg_carry", "k_prequant64", "k_minmax64"])
def test_passes(res, name):
    for k, v in family(res, name).items():
        assert v["waves_per_simd"] >= 4 and v["vgpr_spills"] == 0, (k, v)


# spilled registers and scratch of the launched compression kernels: by rank and
# quantizer (0 grid, 1 point-wise, 2 integers), as measured; none in 1-D
SPILLS = {(3, 0): (4, 104), (3, 1): (6, 56), (3, 2): (41, 200), (2, 0): (0, 0), (2, 1): (6, 32), (2, 2): (34, 144)}
BATCH = {3: (10, 120), 2: (4, 24)}


def test_compression_spills(res):
    for k, v in family(res, "k_compress").items():
        for rank in (1, 2, 3):
            for qm in (0, 1, 2):
                if "ILi%dELb1ELi%dEE" % (rank, qm) in k:
                    n, scratch = SPILLS.get((rank, qm), (0, 0))
                    assert v["vgpr_spills"] <= n and v["scratch_bytes_per_lane"] <= scratch, (k, v)
    for k, v in family(res, "k_batch_compress").items():
        for rank in (1, 2, 3):
            if "ILi%dELb1EE" % rank in k:
                n, scratch = BATCH.get(rank, (0, 0))
                assert v["vgpr_spills"] <= n and v["scratch_bytes_per_lane"] <= scratch, (k, v)
