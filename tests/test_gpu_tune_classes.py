"""What the tuners note.  A grid call whose lanes are (point, time) pairs has no launch shape
to tune and must not settle that of a larger call in the same class (point counts rounded
up to a power of two); the oscillator runs' threshold is the one that runs fastest."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


@pytest.mark.parametrize("small,large,times,charges", [(70000, 120000, 1, 16), (33, 60, 4000, 16)])
def test_a_call_without_a_shape_leaves_its_class_open(tmp_path, monkeypatch, small, large, times, charges):
    import torch
    from paper_2107_12437_amd import lw
    f = tmp_path / "tune.txt"
    monkeypatch.setenv("LW_TUNE_CACHE", str(f))
    monkeypatch.delenv("LW_AUTOTUNE", raising=False)
    g = np.random.default_rng(1)
    ch = I.random_grid_charges(g, charges)
    pts = torch.tensor(I.unit_sphere(g, large).T * 80e-9, device="cuda")
    t = (np.arange(times) + 1) * 1e-15 / times

    def lines():
        return [ln for ln in f.read_text().splitlines() if ln.strip()] if f.exists() else []

    ctx = lw.Context(0)
    try:
        lw.fields(ch, pts[:, :small].contiguous(), t, ctx=ctx)
        before = len(lines())
        lw.fields(ch, pts, t, ctx=ctx)
        torch.cuda.synchronize()
        assert len(lines()) == before + 1              # the larger call's own shape
        lw.fields(ch, pts, t, ctx=ctx)
        assert len(lines()) == before + 1
    finally:
        ctx.close()



COLD = """
import math, sys
import numpy as np
from paper_2107_12437_amd import inputs as I, lw
parts = [I.cluster_dipoles(I.rng_for(90 + k), 12, 40e-9, 10e-9, 2 * math.pi * 200e12, 0.01, True) for k in range(8)]
lw.dipole_run(I.concat_dipoles(parts), (12 * np.arange(9)).astype(np.int32), 1 / 200e12 / 200, 50,
              stepped_min_n="tune", precision=sys.argv[1])
"""


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_run_tuner_in_a_new_process(tmp_path, precision):
    """A process's first trial loads its kernels, which must not count: instances of 12 run
    three times faster per step whole in a workgroup than by launches."""
    f = tmp_path / "tune.txt"
    env = dict(os.environ, LW_TUNE_CACHE=str(f), PYTHONPATH=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    env.pop("LW_AUTOTUNE", None)
    subprocess.run([sys.executable, "-c", COLD, precision], env=env, check=True, timeout=100)
    lines = [ln for ln in f.read_text().splitlines() if ln.startswith("dipoles")]
    assert len(lines) == 1 and int(lines[0].split("|")[1]) > 12, lines


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_run_tuner_knows_which_histories_fit(tmp_path, monkeypatch, precision):
    """12 dipoles with 256 samples (76 KB) run whole in one workgroup, three times faster per
    step than by launches: the threshold must leave them there."""
    import math

    from paper_2107_12437_amd import lw
    f = tmp_path / "tune.txt"
    monkeypatch.setenv("LW_TUNE_CACHE", str(f))
    parts = [I.cluster_dipoles(I.rng_for(90 + k), 12, 40e-9, 10e-9, 2 * math.pi * 200e12, 0.01, True) for k in range(8)]
    off = (12 * np.arange(9)).astype(np.int32)
    ctx = lw.Context(0)
    try:
        lw.dipole_run(I.concat_dipoles(parts), off, 1 / 200e12 / 200, 50, ring_depth=256, stepped_min_n="tune",
                      precision=precision, ctx=ctx)
        lines = [ln for ln in f.read_text().splitlines() if ln.startswith("dipoles")]
        assert len(lines) == 1 and int(lines[0].split("|")[1]) > 12, lines
    finally:
        ctx.close()
