"""Shape classes of the launch-shape tuner next to the sizes that take a launch of their own:
a grid call whose lanes are (point, time) pairs has no shape to tune and must not settle
that of a larger call in the same class (point counts rounded up to a power of two)."""
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
