"""Charges and times that travel as launch arguments against the same call through the
staging buffer (lw_fields_noalloc): equal bits at and about the argument size, outputs and
gradients that do not see the caller's arrays change after the call, and a captured call
whose replays keep the values it was captured with."""
import numpy as np
import pytest

from paper_2107_12437_amd import inputs as I
from tests.helpers import gpu_ready

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_ready(), reason="needs a GPU")]


def workload(nch, nt, npts=200, seed=5):
    g = np.random.default_rng(seed)
    ch = I.random_grid_charges(g, nch)
    pts = (I.unit_sphere(g, npts) * (g.uniform(40e-9, 150e-9, npts))[:, None]).T.copy()
    return ch, pts, (np.arange(nt) + 1) * 3e-16 / nt


# 3,840 bytes: 144 a charge, 8 a time
@pytest.mark.parametrize("nch,nt", [(1, 1), (1, 462), (1, 463), (26, 12), (26, 13), (25, 30), (27, 1), (5, 390), (5, 391)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_arguments_equal_staging(nch, nt, precision):
    import torch
    from paper_2107_12437_amd import lw
    ch, pts, times = workload(nch, nt)
    dp = torch.tensor(pts, device="cuda")
    c = lw.FieldsCall(ch, dp, times.copy(), precision=precision)
    got, fl = c.launch()
    c.times[:] = -1.0                                  # a call has taken its inputs when it returns
    ref, rfl = lw.fields_noalloc(ch, dp, times, precision=precision)
    assert torch.equal(got, ref) and torch.equal(fl, rfl)


def test_captured_call_keeps_its_values():
    import torch
    from paper_2107_12437_amd import lw
    ch, pts, times = workload(5, 7)
    ch2, _, times2 = workload(9, 11, seed=6)
    dp = torch.tensor(pts, device="cuda")
    ctx = lw.Context(0)
    c = lw.FieldsCall(ch, dp, times, precision="fp64", ctx=ctx)
    ref = c.launch()[0].clone()
    other = lw.fields(ch2, dp, times2, precision="fp64")[0].clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        c.launch()
    for _ in range(3):
        c.out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(c.out, ref)
        # the context's own next call, with other inputs
        assert torch.equal(lw.fields(ch2, dp, times2, precision="fp64", ctx=ctx)[0], other)
        torch.cuda.synchronize()
