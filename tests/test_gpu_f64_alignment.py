"""Double fields at any 8-byte alignment: the prequantization's 16-byte loads and
the values behind its last whole group of four, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2304_12557_amd as fz
from oracle import oracle as O
import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("off", [0, 1, 2, 3])
@pytest.mark.parametrize("shape", [(1,), (2,), (3,), (4,), (5,), (1023,), (4097,), (5, 7, 11), (33, 37, 70), (75, 1031), (1_500_003,)])
def test_any_input_alignment(shape, off):
    x = synth.sine_field(shape, seed=5 + len(shape)).astype(np.float64) * 1.000000123
    print("case", shape, off, flush=True)
    n = x.size
    big = torch.full((n + off + 8,), float("nan"), dtype=torch.float64, device="cuda")  # a read past the field would show
    xt = big[off:off + n].view(shape)
    xt.copy_(torch.from_numpy(x))
    for eb, mode, om in ((1e-3, "rel", O.EB_REL), (1e-2, "abs", O.EB_ABS)):
        ref, st = O.compress_f64(x, eb, om, threads=8)
        buf = fz.compress(xt, eb, mode)
        assert st == 0 and fz.stream_info(buf)["status"] == 0
        assert np.array_equal(buf[:fz.stream_size(buf)].cpu().numpy(), ref)
