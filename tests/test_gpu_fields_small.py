"""lw_fields at the sizes its lane-per-(point, time) launch takes and at the edges of that
rule: single points, points that do not fill a wave, charges shared by 1 to 8 waves, every
output group, a masked point, and the sizes just past the rule.  Against the FP64 oracle at
the parity bounds, 1e-12 (FP64) and 1e-5 (mixed) of each output group's magnitude, for B of
the larger of |B| and |E| / c (B = n x E / c cancels where a charge is seen at rest)."""
import numpy as np
import pytest

import oracle as O
from paper_2107_12437_amd import inputs as I
from tests.helpers import GROUPS, gpu_ready

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]

TOL = {"fp64": 1e-12, "mixed": 1e-5}


def workload(npts, nt, nch, seed=4):
    g = np.random.default_rng(seed)
    ch = I.random_grid_charges(g, nch)
    if nch > 4:                                   # every family
        ch["kind"][1], ch["v"][1] = I.UNIFORM_VELOCITY, (0.3 * I.C_LIGHT, 0.1 * I.C_LIGHT, 0.0)
        ch["kind"][2] = I.STATIONARY
    pts = (I.unit_sphere(g, npts) * (g.uniform(40e-9, 150e-9, npts))[:, None]).T.copy()
    return ch, pts, (np.arange(nt) + 1) * 3e-16 / nt


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("npts,nt,nch", [(1, 1, 1), (1, 200, 3), (6, 700, 12), (63, 5, 9), (64, 3, 2), (65, 1, 17),
                                         (1000, 65, 1), (1000, 66, 1), (1000, 97, 3),
                                         (1000, 99, 3), (40, 1700, 2), (41, 1700, 5), (70, 1000, 1)])
def test_sizes_about_the_rule(npts, nt, nch, precision):
    import torch
    from paper_2107_12437_amd import lw
    ch, pts, times = workload(npts, nt, nch)
    dp = torch.tensor(pts, device="cuda")
    out, flags = lw.fields(ch, dp, times, precision=precision)
    torch.cuda.synchronize()
    got = out.double().cpu().numpy()
    ref, rfl = O.fields(ch, pts, times)
    e_c = np.abs(ref[:, 4:7]).max() / I.C_LIGHT
    for name, rows in GROUPS.items():
        size = max(np.abs(ref[:, rows]).max(), e_c if name == "B" else 0.0)
        assert np.abs(got[:, rows] - ref[:, rows]).max() <= TOL[precision] * size, name
    assert np.array_equal(flags.cpu().numpy().astype(np.uint32), np.asarray(rfl).astype(np.uint32))
    # other output groups hold the same bits, and the allocation-free call too
    for sel, rows in ((("E",), slice(4, 7)), (("phi", "B"), [0, 7, 8, 9])):
        o2, _ = lw.fields(ch, dp, times, precision=precision, outputs=sel)
        assert torch.equal(o2, out[:, rows])
    o3, _ = lw.fields(ch, dp, times, precision=precision, outputs=("E", "B", "S"))
    assert torch.equal(o3[:, :6], out[:, 4:])
    S = np.cross(got[:, 4:7], got[:, 7:10], axis=1) * 8.8541878128e-12 * I.C_LIGHT ** 2
    tol = 1e-12 if precision == "fp64" else 1e-6
    assert np.abs(o3[:, 6:].double().cpu().numpy() - S).max() <= tol * np.abs(S).max()
    if nch * nt * 272 < (3 << 20):
        o4, f4 = lw.fields_noalloc(ch, dp, times, precision=precision)
        assert torch.equal(o4, out) and torch.equal(f4, flags)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_masked_points_at_single_times(precision):
    """A point on a stationary charge (masked at every time) and one that a moving charge
    passes at one time only: NaN there, the flag on the point, other times untouched."""
    import torch
    from paper_2107_12437_amd import lw
    ch = I.empty_charges(9)
    ch["q"][:] = I.E_CHARGE
    ch["c0"][:, 0] = np.arange(9) * 20e-9
    ch["kind"][4], ch["v"][4] = I.UNIFORM_VELOCITY, (0.0, 0.2 * I.C_LIGHT, 0.0)
    times = np.array([0.0, 1e-16, 2e-16])
    pts = np.array([[0.0, 0.0, 0.0], [80e-9, 0.2 * I.C_LIGHT * 1e-16, 0.0], [30e-9, 5e-9, 7e-9]]).T.copy()
    out, flags = lw.fields(ch, torch.tensor(pts, device="cuda"), times, precision=precision)
    torch.cuda.synchronize()
    nan = torch.isnan(out).all(dim=1).cpu().numpy()
    assert flags.cpu().tolist() == [1, 1, 0]
    assert nan.tolist() == [[True, False, False], [True, True, False], [True, False, False]]
    assert np.isfinite(out.cpu().numpy()[:, :, 2]).all()
