"""The stepped path's units of targets x sources (more than 2,048 fixed targets and 5,500 rounds of 64
sources here) at the edges of its layout: instances about 64 and 128 targets and about
whole source chunks, sizes that leave a last tile partly filled, one larger than many chunks,
long light times (smaller tiles) and ones past the tiles' reach, offsets outside the series'
range, the pre-history's end.  Against the oracle, and against each instance alone, which
takes the launch of few targets; both at the suite's bounds.  Runs in parts have equal bits."""
import math

import numpy as np
import pytest
import torch

from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready
from tests.test_gpu_dipole import assert_state_close, gpu_run, oracle_run

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

CDT = I.C_LIGHT / 200e12 / 200


def batch(sizes, steps, moment=1e-12, half=100e-9, sep=9e-9, seed=8):
    g = I.rng_for(seed)
    parts = []
    for n in sizes:
        d = I.cluster_dipoles(g, n, half, sep, 2 * math.pi * 200e12, 0.01, True)
        d["d0"][:] = I.E_CHARGE * moment * (-1.0) ** np.arange(n) * np.linspace(0.2, 1.0, n)
        parts.append(d)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    return {"dipoles": I.concat_dipoles(parts), "inst_off": off, "dt": 1 / 200e12 / 200, "steps": steps}


def part(w, k, steps=None):
    a, b = w["inst_off"][k], w["inst_off"][k + 1]
    return dict(w, dipoles={q: np.asarray(v)[a:b] for q, v in w["dipoles"].items()},
                inst_off=np.array([0, b - a], np.int32), steps=steps or w["steps"])


def check(got, ref, w, precision, what):
    if precision == "fp64":
        assert_state_close(got, ref, w, what=what)
    else:
        assert_state_close(got, ref, w, keys=("d", "d_dot", "energy"), tol=1e-5, what=what)


SIZES = [670, 300, 300, 200, 129, 128, 127, 97, 65, 64, 33]    # 2,113 targets


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("moment,half", [(1e-12, 100e-9), (4e-11, 100e-9), (1e-12, 500e-9), (1e-12, 2.3e-6)])
def test_against_instances_alone(moment, half, precision):
    # half 100 nm to 2.3 um: light times up to 46, 230 and 1,060 steps (tiles of 16, 4, none)
    w = batch(SIZES, 50, moment, half)
    got = gpu_run(w, "strict", precision=precision, energy_balance=True)
    for k, n in enumerate(SIZES):
        a, b = w["inst_off"][k], w["inst_off"][k + 1]
        alone = gpu_run(part(w, k), "strict", precision=precision, energy_balance=True)
        check({q: v[:, a:b] for q, v in got.items()}, alone, part(w, k), precision, f"{n} dipoles")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_against_the_oracle(precision):
    w = batch(SIZES, 45)
    got = gpu_run(w, "extrapolate", precision=precision)
    for k in (8, 10):
        a, b = w["inst_off"][k], w["inst_off"][k + 1]
        check({q: v[:, a:b] for q, v in got.items()}, oracle_run(part(w, k), "extrapolate", extended=True), part(w, k),
              precision, f"{SIZES[k]} dipoles")


def test_runs_in_parts_and_strides():
    from paper_2107_12437_amd import lw
    w = batch(SIZES, 50)
    kw = dict(precision="fp64", energy_balance=True)
    whole = gpu_run(w, "strict", **kw)
    state = lw.dipole_state(w["dipoles"], w["inst_off"], w["dt"])
    a = lw.dipole_run(w["dipoles"], w["inst_off"], w["dt"], 21, state=state, **kw)
    b = lw.dipole_run(w["dipoles"], w["inst_off"], w["dt"], 29, state=state, resume=True, **kw)
    torch.cuda.synchronize()
    third = gpu_run(w, "strict", stride=3, **kw)
    for q in whole:
        assert np.array_equal(whole[q], np.concatenate([a[q].cpu().numpy(), b[q].cpu().numpy()[1:]])), q
        assert np.array_equal(whole[q][::3], third[q]), q
