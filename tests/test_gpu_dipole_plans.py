"""The kernels of oscillator runs by their numbers of targets, sources and instances, against
the FP64 oracle across the edges of each choice: launches per step (few targets, some
with few or many sources each, many) and instances held whole (few or many)."""
import math

import numpy as np
import pytest

import oracle as O
from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready
from tests.test_gpu_dipole import TOL_MIXED_STATE, assert_state_close

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

DT = 1 / 200e12 / 200


def batch(n, count):
    """`count` instances of n, of which the first and the last differ from the rest."""
    half = 9e-9 * n ** (1 / 3)                 # light times of up to about 5 n^(1/3) / 2 steps
    parts = [I.cluster_dipoles(I.rng_for(60 + k), n, half, 10e-9, 2 * math.pi * 200e12, 0.01, True) for k in range(3)]
    pick = [0] + [1] * (count - 2) + [2] if count > 1 else [0]
    return I.concat_dipoles([parts[k] for k in pick]), (n * np.arange(count + 1)).astype(np.int32), parts


# targets: up to 512, 513 to 1,024 with up to 128 other dipoles each or more, over 1,024 with a
# wave or (4,500 rounds of 64 sources, up to 2,048 targets) a workgroup each
@pytest.mark.parametrize("n,count", [(16, 32), (16, 33), (129, 4), (130, 4), (130, 3), (257, 1), (258, 1), (258, 2),
                                     (16, 64), (16, 65), (200, 8)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_targets_and_sources_about_the_plans_edges(precision, n, count):
    """The first and the last instance as the oracle has them alone (instances do not act on
    each other), at the run tests' tolerances."""
    from paper_2107_12437_amd import lw
    dip, off, parts = batch(n, count)
    steps = 60 if n == 16 else 24 if n <= 130 else 12
    r = lw.dipole_run(dip, off, DT, steps, out_stride=4, precision=precision, stepped_min_n=2)
    for part, lo in ((parts[0], 0), (parts[2], (count - 1) * n))[:count]:
        got = {k: v.cpu().numpy()[:, lo:lo + n] for k, v in r.items()}
        w = {"dipoles": part, "inst_off": [0, n]}
        ref = O.dipole_run(part, [0, n], DT, steps, out_stride=4)
        if precision == "fp64":
            assert_state_close(got, ref, w, what=f"{count} x {n}")
        else:
            assert_state_close(got, ref, w, keys=("d", "d_dot", "energy"), tol=TOL_MIXED_STATE, what=f"{count} x {n}")


@pytest.mark.parametrize("n,count", [(5, 3071), (5, 3072), (10, 1535), (10, 1536), (16, 1536)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_many_instances_held_whole(precision, n, count):
    """The kernel with a lane per pair, and the general one where instances are many."""
    from paper_2107_12437_amd import lw
    dip, off, parts = batch(n, count)
    steps = 100
    r = lw.dipole_run(dip, off, DT, steps, out_stride=20, precision=precision, stepped_min_n=-1)
    for part, lo in ((parts[0], 0), (parts[2], (count - 1) * n)):
        got = {k: v.cpu().numpy()[:, lo:lo + n] for k, v in r.items()}
        w = {"dipoles": part, "inst_off": [0, n]}
        ref = O.dipole_run(part, [0, n], DT, steps, out_stride=20)
        if precision == "fp64":
            assert_state_close(got, ref, w, what=f"{count} x {n}")
        else:
            assert_state_close(got, ref, w, keys=("d", "d_dot", "energy"), tol=TOL_MIXED_STATE, what=f"{count} x {n}")


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_segment_edges_in_the_general_kernel(precision):
    """The series drives' segment edges and range limits (test_gpu_dipole_series) in instances
    too large for the kernels with a lane per pair: a pair and 16 far dipoles each."""
    from tests import test_gpu_dipole_series as S
    seps = [S.CDT * m * (1 + e) for m in (0.5, 1.0, 2.0, 7.0) for e in (-4e-5, 0.0, 3e-5)]
    w = S.pairs(seps, [1e-13, 1e-12, 4e-12, 4e-11], 100)
    g = np.random.default_rng(3)
    parts = []
    for k in range(0, len(seps), 2):
        far = I.cluster_dipoles(g, 16, 60e-9, 12e-9, 2 * math.pi * 200e12, 0.01, True)
        far["origin"][:, 1] += 300e-9
        parts += [{q: np.asarray(v)[2 * k:2 * k + 2] for q, v in w["dipoles"].items()}, far]
    w = dict(w, dipoles=I.concat_dipoles(parts), inst_off=np.arange(0, 18 * (len(parts) // 2) + 1, 18, dtype=np.int32))
    got = S.gpu_run(w, "extrapolate", precision=precision, stepped_min_n=-1)
    ref = S.oracle_run(w, "extrapolate")
    if precision == "fp64":
        assert_state_close(got, ref, w)
    else:
        assert_state_close(got, ref, w, keys=("d", "d_dot", "energy"), tol=TOL_MIXED_STATE)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("moment", [1e-12, 4e-11])
def test_tiles_of_four_sources(precision, moment):
    """Light times of 300 steps leave room for four sources' windows; the larger moment puts
    sources of every round outside the series' range."""
    from tests import test_gpu_dipole_tile as T
    w = T.batch(T.SIZES, 30, moment, 720e-9)
    got = T.gpu_run(w, "strict", precision=precision)
    for k in (0, 4, 6, 9, 10):
        a, b = w["inst_off"][k], w["inst_off"][k + 1]
        alone = T.gpu_run(T.part(w, k), "strict", precision=precision)
        T.check({q: v[:, a:b] for q, v in got.items()}, alone, T.part(w, k), precision, f"{T.SIZES[k]} dipoles")
