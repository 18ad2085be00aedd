"""Hand-out of chunk tickets inside a compression workgroup.

Thread 0 takes the tickets, the other waves read them from LDS.  A wave may
read the first ticket late (nothing holds it between the barrier after the
hand-out and its read), while thread 0 goes on to leave the next ticket with no
barrier before that: the two must not share a word.  A workgroup whose first
field failed its range pass leaves the next ticket at once, so the batch test
runs many such fields.
"""
import os
import re

import numpy as np
import pytest

import paper_2304_12557_amd as fz
from oracle import oracle as O
import synth

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_12557_amd", "csrc")


@pytest.mark.parametrize("name,kernel", [("fz_compress.hip", "k_compress"), ("fz_batch.hip", "k_batch_compress")])
def test_first_ticket_has_its_own_word(name, kernel):
    src = open(os.path.join(CSRC, name)).read()
    body = src[re.search(r"void %s\(" % kernel, src).start():]
    body = body[:body.index("\n}\n")]
    loop = re.search(r"\n    for \(;;", body).start()
    first = re.findall(r"S\.(\w+) = atomicAdd\(", body[:loop])
    after_barrier = re.findall(r"readfirstlane\(\(uint32_t\)S\.(\w+)\)", body[:loop])
    assert first and first == after_barrier
    assert not re.search(r"S\.%s\b" % first[0], body[loop:])  # not written (nor read) once the loop runs


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(5,), (3, 70), (2, 3, 5)])
def test_skipped_fields(shape):
    import torch

    n = 900  # more chunks than workgroups
    xs = []
    for i in range(n):
        x = synth.sine_field(shape, seed=100 + i)
        if i % 7:  # the range pass fails: its chunk is skipped
            x.reshape(-1)[i % x.size] = np.nan
        xs.append(x)
    ts = [torch.from_numpy(x).cuda() for x in xs]
    outs = [torch.zeros(fz.compress_bound(shape), dtype=torch.uint8, device="cuda") for _ in xs]
    b = fz.Batch.compress([(t, 1e-3, "rel", o) for t, o in zip(ts, outs)])
    for run in range(5):
        b.run()
        torch.cuda.synchronize()
        print("run", run, shape, flush=True)
        for i in range(n):
            info = fz.stream_info(outs[i])
            assert info["status"] == (1 if i % 7 else 0), (run, i)
            if i % 7 == 0 and run in (0, 4):
                ref, st = O.compress(xs[i], 1e-3, O.EB_REL)
                assert st == 0 and np.array_equal(outs[i][:fz.stream_size(outs[i])].cpu().numpy(), ref), (run, i)
    b.close()
