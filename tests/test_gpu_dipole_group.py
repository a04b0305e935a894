"""The one-workgroup kernel of instances with 5 to 16 fixed dipoles, at the edges of its
layout (8 or 16 lanes per target, a last wave with one target) and of its rules (series
range, segment crossings, batches that mix every kernel), against the oracle's extended build
at the suite's bounds; runs in parts and runs beside other instances against the same bits."""
import math

import numpy as np
import pytest
import torch

from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready
from tests.test_gpu_dipole import assert_state_close, gpu_run, oracle_run

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

CDT = I.C_LIGHT / 200e12 / 200


def batch(sizes, steps, moment=1e-12, seed=6, sep=10e-9):
    """One cluster per size; in each, dipole 1 stands a whole number of light steps (to 3e-5)
    from dipole 0 along z, and moments alternate in sign."""
    g = I.rng_for(seed)
    parts = []
    for n in sizes:
        d = I.cluster_dipoles(g, n, 30e-9 * max(1.0, n / 4) ** (1 / 3), sep, 2 * math.pi * 200e12, 0.01, True)
        if n > 1:
            d["origin"][1] = d["origin"][0] + np.array([0.0, 0.0, 31 * CDT * (1 + 3e-5)])
        d["d0"][:] = I.E_CHARGE * moment * (-1.0) ** np.arange(n) * np.linspace(0.2, 1.0, n)
        parts.append(d)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    return {"dipoles": I.concat_dipoles(parts), "inst_off": off, "dt": 1 / 200e12 / 200, "steps": steps}


def check(got, w, policy, precision, what):
    ref = oracle_run(w, policy, extended=True)
    if precision == "fp64":
        assert_state_close(got, ref, w, what=what)
    else:
        assert_state_close(got, ref, w, keys=("d", "d_dot", "energy"), tol=1e-5, what=what)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("sizes,moment,sep", [([5], 1e-12, 10e-9), ([8], 1e-12, 10e-9), ([9], 4e-11, 10e-9),
                                              ([10], 1e-12, 10e-9), ([15], 1e-13, 10e-9), ([16], 1e-12, 10e-9),
                                              ([16, 5, 12, 9], 1e-12, 10e-9), ([7, 13], 1e-12, 6.4e-9)])
def test_sizes(sizes, moment, sep, precision):
    w = batch(sizes, 60, moment, sep=sep)
    policy = "strict" if sep > 8e-9 else "extrapolate"
    check(gpu_run(w, policy, precision=precision, stepped_min_n=-1), w, policy, precision, str(sizes))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_of_every_kernel(precision):
    # one wave, this kernel, the general persistent kernel and (default rule) the stepped one
    w = batch([3, 18, 6, 1, 14, 4, 16], 40)
    for kw in ({}, {"stepped_min_n": -1}, {"stepped_min_n": 7}):
        got = gpu_run(w, "strict", precision=precision, energy_balance=True, **kw)
        check(got, w, "strict", precision, str(kw))
    alone = batch([3, 18, 6], 40)
    other = gpu_run(alone, "strict", precision=precision, energy_balance=True)
    full = gpu_run(w, "strict", precision=precision, energy_balance=True)
    k = slice(21, 27)
    for q in full:
        assert np.array_equal(other[q][:, k], full[q][:, k]), q


@pytest.mark.parametrize("n,ring", [(5, 0), (12, 0), (12, 256)])
def test_runs_in_parts(n, ring):
    from paper_2107_12437_amd import lw
    w = batch([n], 90)
    kw = dict(precision="fp64", energy_balance=True, ring_depth=ring)
    whole = gpu_run(w, "strict", **kw)
    state = lw.dipole_state(w["dipoles"], w["inst_off"], w["dt"], ring_depth=ring)
    a = lw.dipole_run(w["dipoles"], w["inst_off"], w["dt"], 37, state=state, **kw)
    b = lw.dipole_run(w["dipoles"], w["inst_off"], w["dt"], 53, state=state, resume=True, **kw)
    torch.cuda.synchronize()
    for q in whole:
        parts = np.concatenate([a[q].cpu().numpy(), b[q].cpu().numpy()[1:]])
        assert np.array_equal(whole[q], parts), q


def test_stop_on_the_speed_limit():
    # every wave leaves at the same step, the error is reported, other instances finish
    from paper_2107_12437_amd import lw
    w = batch([12, 6], 50)
    free = gpu_run(w, "strict")
    top = np.abs(free["d_dot"][:, :12]).max(axis=0) / I.E_CHARGE
    first = int(np.argmax(np.abs(free["d_dot"][:, :12]).max(axis=1) / I.E_CHARGE * 1.0 > 0.5 * top.max()))
    d = w["dipoles"]
    vfac = np.maximum(d["m1"], d["m2"]) / (d["m1"] + d["m2"]) / d["q"]
    limit = float((vfac[:12, None].T * np.abs(free["d_dot"][first - 1, :12])).max()) * 1.0000001
    ctx = lw.Context(0)
    r = lw.dipole_run(d, w["inst_off"], w["dt"], 50, max_vel=limit, check=False, ctx=ctx)
    torch.cuda.synchronize()
    assert np.array_equal(r["d"][:first, :12].cpu().numpy(), free["d"][:first, :12])
    with pytest.raises(lw.LWError):
        lw._check(lw.load_library().lw_sync_status(ctx.handle, None))
