"""A stepped run's launches, one by one or as graphs of 64 or 256 steps by its length: the
lengths about the rule and with a remainder, against the same run in parts below it, equal
bits, at every step and at a stride."""
import math

import numpy as np
import pytest
import torch

from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready
from tests.test_gpu_dipole import gpu_run

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.mark.parametrize("steps,stride", [(383, 1), (384, 1), (455, 7), (4095, 9), (4100, 10)])
def test_lengths_about_the_rule(steps, stride):
    from paper_2107_12437_amd import lw
    d = I.cluster_dipoles(I.rng_for(4), 20, 60e-9, 10e-9, 2 * math.pi * 200e12, 0.01, True)
    w = {"dipoles": d, "inst_off": np.array([0, 20], np.int32), "dt": 1 / 200e12 / 200, "steps": steps}
    whole = gpu_run(w, "strict", stride=stride)
    state = lw.dipole_state(d, w["inst_off"], w["dt"])
    last, done = {}, 0
    while done < steps:
        k = min(steps - done, 315)               # a multiple of every stride here but 10
        k -= k % stride if done + k < steps else 0
        r = lw.dipole_run(d, w["inst_off"], w["dt"], k, out_stride=stride, state=state, resume=done > 0)
        torch.cuda.synchronize()
        for q, v in r.items():
            v = v.cpu().numpy()
            a = done // stride
            assert np.array_equal(whole[q][a:a + len(v)], v), (q, done)
        done += k
    assert done == steps
