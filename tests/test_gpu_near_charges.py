"""Grid fields close to the charges, where the retarded-time problem is quasi-static, and at
high speeds, where it is far from quadratic: points at a stated distance from a charge's
retarded position, so that every point's light time and 1 - n.beta are known.  Against the
extended-precision oracle, each point relative to its own field (B to the larger of |B|
and |E| / c: B = n x E / c cancels to beta times that for slow charges), at the parity
bounds 1e-12 (FP64) and 1e-5 (mixed) plus rounding: the coordinates and the phase carry
errors of a few eps times the orbit's size and the phase, which the field takes up by
at most (1 + beta / kappa) (1 + 3 beta / kappa); the mixed path's FP32 terms carry 2^-24."""
import math

import numpy as np
import pytest

import oracle as O
from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

EPS = 2.0 ** -53
TOL = {"fp64": 1e-12, "mixed": 1e-5}
PRECISIONS = pytest.mark.parametrize("precision", ["fp64", "mixed"])
KINDS = pytest.mark.parametrize("kind", [I.CIRCULAR, I.LINEAR_OSC])


def near_orbit(kind, beta, dist, n=203, seed=0, omega=2 * math.pi * 200e12):
    """One charge, a time, n points `dist` amplitudes from its retarded position (not a
    multiple of the wave), their kappa and the size of the rounding in their coordinates."""
    g = np.random.default_rng((seed, kind, int(1e6 * beta), int(1e3 * dist)))
    ch = I.empty_charges(1)
    e1, e2 = I.orbit_basis(g.normal(size=3))
    amp, phase, t = beta * I.C_LIGHT / abs(omega), g.uniform(0, 2 * math.pi), g.uniform(-2e-14, 2e-14)
    ch["kind"][:], ch["q"][:], ch["amp"][:], ch["omega"][:], ch["phase"][:] = kind, I.E_CHARGE, amp, omega, phase
    ch["e1"][0], ch["e2"][0] = e1, e2
    th = omega * (t - dist * amp / I.C_LIGHT) + phase
    pos, vel = amp * math.cos(th) * e1, -amp * omega / I.C_LIGHT * math.sin(th) * e1
    if kind == I.CIRCULAR:
        pos, vel = pos + amp * math.sin(th) * e2, vel + amp * omega / I.C_LIGHT * math.cos(th) * e2
    d = I.unit_sphere(g, n)
    scale = (1.0 + 1.0 / dist) * (1.0 + abs(omega * t) + abs(th))
    return ch, t, (pos + dist * amp * d).T.copy(), 1.0 - d @ vel, scale


def errors(got, ref):
    """Largest relative error of each point's Phi, A, E and B, each against its own size."""
    e_c = np.linalg.norm(ref[4:7], axis=0) / I.C_LIGHT
    worst = np.abs(got[0] - ref[0]) / np.abs(ref[0])
    for rows, floor in ((slice(1, 4), np.abs(ref[0]) / I.C_LIGHT), (slice(4, 7), 0.0 * e_c), (slice(7, 10), e_c)):
        size = np.maximum(np.linalg.norm(ref[rows], axis=0), floor)
        worst = np.maximum(worst, np.linalg.norm(got[rows] - ref[rows], axis=0) / size)
    return worst


def bounds(precision, beta, kappa, scale):
    lift = (1.0 + beta / kappa) * (1.0 + 3.0 * beta / kappa)
    tol = TOL[precision] + 8.0 * EPS * scale * lift
    return tol if precision == "fp64" else tol + 8.0 * 2.0 ** -24 * lift


def gpu_fields(ch, pts, t, precision):
    import torch
    from paper_2107_12437_amd import lw
    out, flags = lw.fields(ch, torch.tensor(pts, device="cuda"), np.array([t]), precision=precision, mask_radius=0.0)
    torch.cuda.synchronize()
    assert not flags.any()
    return out[0].double().cpu().numpy()


def check(case, beta, precision):
    ch, t, pts, kappa, scale = case
    ref = O.fields(ch, pts, [t], mask_radius=0.0, extended=True)[0][0]
    worst, tol = errors(gpu_fields(ch, pts, t, precision), ref), bounds(precision, beta, kappa, scale)
    assert np.isfinite(worst).all()
    i = int((worst / tol).argmax())
    assert worst[i] <= tol[i], (worst[i], tol[i], kappa[i])


@KINDS
@PRECISIONS
@pytest.mark.parametrize("beta", [0.3, 0.6, 0.7, 0.9, 0.98])
@pytest.mark.parametrize("dist", [1.5, 4.0])
def test_phase_rotation_over_its_range(kind, precision, beta, dist):
    """The retarded phase lies up to beta + pi / 128 from the start's, through which the
    solve turns by polynomials."""
    check(near_orbit(kind, beta, dist), beta, precision)


@KINDS
@PRECISIONS
@pytest.mark.parametrize("beta", [1e-6, 1e-3, 3e-3, 0.01, 0.03, 0.1, 0.3, 0.6, 0.9, 0.99])
def test_near_orbits(kind, precision, beta):
    """Next to the charge and about its orbit, where the light time is far below a radian
    of phase for all but the fastest; either sense of rotation."""
    for k, dist in enumerate((0.02, 0.1, 0.3, 0.5, 1.0, 2.0)):
        check(near_orbit(kind, beta, dist, omega=(-1) ** k * 2 * math.pi * 200e12), beta, precision)
        check(near_orbit(kind, beta, dist, omega=-(-1) ** k * 2 * math.pi * 200e12, n=70), beta, precision)


@PRECISIONS
@pytest.mark.parametrize("beta", [0.95, 0.99])
def test_fast_oscillation_has_one_root(precision, beta):
    """Where the solve's function has inflections next to no root of it: a step from there
    can be small."""
    for dist in (0.5, 1.0, 1.5):
        check(near_orbit(I.LINEAR_OSC, beta, dist, n=20011), beta, precision)


@PRECISIONS
@pytest.mark.parametrize("beta,dist", [(2e-4, 0.02), (0.82, 0.02), (0.93, 0.011), (0.99, 0.023)])
def test_bracket_next_to_an_orbit(precision, beta, dist):
    """Points whose solve ends in the safeguarded solver, seen across the motion (kappa = 1),
    where the orbit's nearest point is the charge itself: the bracket's end lies at the root
    but for its own rounding."""
    check(near_orbit(I.CIRCULAR, beta, dist, n=20011), beta, precision)


@KINDS
@pytest.mark.parametrize("beta,dist", [(1e-3, 0.1), (0.01, 0.3), (0.03, 0.5), (0.1, 0.3)])
def test_gradient_near_orbits(kind, beta, dist):
    """The gradients take the same solve: against automatic differentiation in torch FP64,
    to 1e-10 of the parameter's largest gradient (as the other families' test)."""
    import torch
    from tests import test_gpu_adjoint_families as F
    ch, t, pts, _, _ = near_orbit(kind, beta, dist, n=81)
    cot = F.cotangent(1, pts.shape[1], ("E",))
    from paper_2107_12437_amd import lw
    got = lw.fields_vjp(ch, torch.tensor(pts, device="cuda"), np.array([t]), torch.tensor(cot, device="cuda"),
                        outputs=("E",), mask_radius=0.0).cpu().numpy()
    F.assert_close(got, F.reference(ch, pts, [t], torch.tensor(cot), ("E",), "total"), 1e-10)


def near_acceleration(speed, share, n, t=1e-15, seed=0):
    """One charge accelerated from rest to `speed` c at time t, n points on its light sphere
    of emission time `share` t; as near_orbit."""
    g = np.random.default_rng((seed, int(1e6 * speed), int(1e6 * share)))
    ch = I.empty_charges(1)
    e1 = I.unit_sphere(g, 1)[0]
    acc, tp = speed * I.C_LIGHT / t, share * t
    ch["kind"][:], ch["q"][:], ch["accel"][:], ch["e1"][0] = I.ACCEL, I.E_CHARGE, acc, e1
    d = I.unit_sphere(g, n)
    pts = (0.5 * acc * tp * tp * e1 + I.C_LIGHT * (t - tp) * d).T.copy()
    return ch, t, pts, 1.0 - share * speed * (d @ e1), 1.0 + 1.0 / (1.0 - share)


@PRECISIONS
@pytest.mark.parametrize("speed", [1e-3, 0.3, 0.6, 0.8, 0.9, 0.99])
def test_near_an_accelerated_charge(precision, speed):
    """From points that see it just started to points within 0.001 c t of it: behind a fast
    one the solve's polynomial has other roots and inflections."""
    for share in (0.02, 0.3, 0.4, 0.5, 0.6, 0.7, 0.8, 0.9, 0.95, 0.99, 0.999):
        check(near_acceleration(speed, share, n=20011), speed * share, precision)
