"""The retarded-time solves of the grid kernels where their rules change: the near-field
start (|omega tau| around 15 steps of the phase grid), frequencies down to zero and of
either sign, phases of many turns, high speeds (lanes that fall back), points about the
light sphere of an accelerated charge's start, and the uniform-velocity form's switch at
|v| = 0.999 c.  Against the FP64 oracle at the parity bounds, 1e-12 (FP64) and 1e-5 (mixed)
of each output group's magnitude, for B of the larger of |B| and |E| / c (B = n x E / c
cancels to beta times that for slow charges), plus what a phase rounding of 4 eps |omega
tau| on either side does to a field that varies as kappa^-3."""
import math

import numpy as np
import pytest

import oracle as O
from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

TOL = {"fp64": 1e-12, "mixed": 1e-5}


def shell(radius, n=203, seed=5):
    """n points (not a multiple of the wave) around the origin, radii within 20 % of `radius`."""
    g = np.random.default_rng(seed)
    return (I.unit_sphere(g, n) * (radius * g.uniform(0.8, 1.2, n))[:, None]).T.copy()


def check(ch, pts, times, precision, phase, beta=0.0):
    import torch
    from paper_2107_12437_amd import lw
    out, flags = lw.fields(ch, torch.tensor(pts, device="cuda"), times, precision=precision)
    torch.cuda.synchronize()
    assert not flags.any()
    got = out.double().cpu().numpy()
    ref, _ = O.fields(ch, pts, times)
    tol = TOL[precision] + 4.0 * 2.2e-16 * phase * (1.0 + 3.0 * beta / (1.0 - beta))
    e_c = np.abs(ref[:, 4:7]).max() / I.C_LIGHT
    for name, rows in (("phi", slice(0, 1)), ("A", slice(1, 4)), ("E", slice(4, 7)), ("B", slice(7, 10))):
        r, d = ref[:, rows], got[:, rows] - ref[:, rows]
        assert np.isfinite(got[:, rows]).all(), name
        size = max(np.abs(r).max(), e_c if name == "B" else 0.0)
        assert np.abs(d).max() <= tol * size, (name, np.abs(d).max() / size, tol)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", [I.CIRCULAR, I.LINEAR_OSC])
@pytest.mark.parametrize("turns", [0.0, 1e-9, 1e-3, 0.1, 0.117, 0.25, 3.0, 4e4])
@pytest.mark.parametrize("beta", [1e-6, 0.3, 0.85])
def test_orbits_over_phase_and_speed(precision, kind, turns, beta):
    dist = 40e-9
    omega = 2 * math.pi * turns * I.C_LIGHT / dist
    ch = I.empty_charges(2)
    ch["kind"][:] = kind
    ch["q"][:] = (I.E_CHARGE, -0.7 * I.E_CHARGE)
    ch["c0"][1] = (3e-9, -2e-9, 1e-9)
    e1, e2 = I.orbit_basis(np.array([0.3, -0.5, 0.8]))
    ch["e1"][:], ch["e2"][:] = e1, e2
    # the orbit stays inside a fifth of the distance
    ch["amp"][:] = min(beta * I.C_LIGHT / omega, 0.2 * dist) if omega > 0 else 0.2 * dist
    ch["omega"][:] = (omega, -omega)
    ch["phase"][:] = (0.4, -2.0)
    times = np.array([-2e-16, 0.0, 7e-16])
    # times are a few femtoseconds: their own phase rounds like the light time's
    check(ch, shell(dist), times, precision, 2 * math.pi * turns * 1.3 + abs(omega) * 7e-16, beta)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("speed", [1e-6, 0.3, 0.6, 0.9])
def test_acceleration_about_the_start(precision, speed):
    """Points on either side of |x - c0| = c t, where the charge is seen at rest or moving."""
    t = 4e-16
    ch = I.empty_charges(1)
    ch["kind"][:], ch["q"][:], ch["accel"][:] = I.ACCEL, I.E_CHARGE, speed * I.C_LIGHT / t
    ch["e1"][0] = I.unit_sphere(np.random.default_rng(2), 1)[0]
    # clear of the sphere itself (where either reading of the start is within rounding) and
    # of the charge's own path
    pts = np.concatenate([shell(I.C_LIGHT * t * f, n=67, seed=k) for k, f in enumerate((0.9, 1.3, 4.0))], axis=1)
    pts = pts[:, np.linalg.norm(pts, axis=0) > 0.75 * I.C_LIGHT * t]
    times = np.array([-1e-16, 0.0, 0.5 * t, t])
    check(ch, pts, times, precision, 0.0)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("beta", [0.5, 0.9989, 0.9991, 0.99999])
def test_uniform_velocity_on_either_side_of_its_switch(precision, beta):
    ch = I.empty_charges(1)
    ch["kind"][:], ch["q"][:] = I.UNIFORM_VELOCITY, I.E_CHARGE
    ch["v"][0] = beta * I.C_LIGHT * I.unit_sphere(np.random.default_rng(3), 1)[0]
    pts = shell(50e-9)
    # beta^2 is rounded to FP32 per point in the mixed field terms: 1 - n.beta keeps
    # 2^-24 / (1 - beta) of its value there
    import torch
    from paper_2107_12437_amd import lw
    if precision == "mixed" and beta > 0.99:
        out, _ = lw.fields(ch, torch.tensor(pts, device="cuda"), np.array([1e-16]), precision="mixed")
        ref, _ = O.fields(ch, pts, np.array([1e-16]))
        got = out.double().cpu().numpy()
        assert np.isfinite(got).all()
        assert np.abs(got[:, 0] - ref[:, 0]).max() <= 8 * 2.0 ** -24 / (1 - beta) * np.abs(ref[:, 0]).max()
        return
    check(ch, pts, np.array([-1e-16, 1e-16]), precision, 0.0 if beta < 0.99 else 1.0 / (1 - beta) ** 2)
