"""The oscillator drive's series path (small offsets, closed forms on stored segments) at
the edges of its rules, against the oracle's extended build at the suite's bounds: charges
whose retarded time crosses a stored step (separations within 1e-4 of a multiple of c dt),
offsets and speeds on either side of the series' range, the end of the static pre-history,
and the newest sample under the extrapolating policy; on the one-wave kernel, the general
persistent kernel, the launch of few targets and the one-wave-per-target launch."""
import math

import numpy as np
import pytest

from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready
from tests.test_gpu_dipole import assert_state_close, gpu_run, oracle_run

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

CDT = I.C_LIGHT / 200e12 / 200


def pairs(seps, moments, steps, axis_spread=True):
    w = I.workload_dipole_pairs(seps=np.asarray(seps, dtype=float), steps=steps)
    d = w["dipoles"]
    g = np.random.default_rng(7)
    if axis_spread:
        d["axis"][:] = I.unit_sphere(g, len(d["omega0"]))
    d["d0"][0::2] = I.E_CHARGE * np.resize(moments, len(seps))
    d["d0"][1::2] = -0.3 * d["d0"][0::2]
    return w


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("path", ["small", "general", "wide", "wave"])
def test_segment_edges_and_range_limits(path, precision):
    # separations at and about whole and half steps of light, two beyond them
    seps = [CDT * m * (1 + e) for m in (0.5, 1.0, 1.5, 2.0, 7.0) for e in (-4e-5, 0.0, 3e-5)] + [3.3e-9, 260e-9]
    # offsets of 5e-14 to 2e-11 m: 1e-6 to 2^-8 of these separations, speeds to 4e-5 c
    moments = [1e-13, 1e-12, 4e-12, 4e-11]
    w = pairs(seps, moments, 150)
    n = len(seps)
    if path == "wave":                       # more than 1,024 targets
        reps = 1200 // (2 * n) + 1
        w = dict(w, dipoles=I.concat_dipoles([w["dipoles"]] * reps),
                 inst_off=np.arange(0, 2 * n * reps + 1, 2, dtype=np.int32))
    kw = {"small": {}, "general": {}, "wide": {"stepped_min_n": 2}, "wave": {"stepped_min_n": 2}}[path]
    if path == "general":                    # a third, far dipole in each instance of five
        g = np.random.default_rng(3)
        parts = []
        for k in range(0, n, 3):
            far = I.cluster_dipoles(g, 3, 60e-9, 12e-9, 2 * math.pi * 200e12, 0.01, True)
            far["origin"][:, 1] += 300e-9
            parts += [{q: np.asarray(v)[2 * k:2 * k + 2] for q, v in w["dipoles"].items()}, far]
        w = dict(w, dipoles=I.concat_dipoles(parts), inst_off=np.arange(0, 5 * (len(parts) // 2) + 1, 5, dtype=np.int32))
    got = gpu_run(w, "extrapolate", precision=precision, **kw)
    if path == "wave":
        for k in range(1, reps):             # equal instances, equal bits
            assert np.array_equal(got["d"][:, :2 * n], got["d"][:, 2 * n * k:2 * n * (k + 1)])
        w = pairs(seps, moments, 150)
        got = {q: v[:, :2 * n] for q, v in got.items()}
    ref = oracle_run(w, "extrapolate", extended=True)
    if precision == "fp64":
        assert_state_close(got, ref, w, what=path)
    else:
        assert_state_close(got, ref, w, keys=("d", "d_dot", "energy"), tol=1e-5, what=path)
