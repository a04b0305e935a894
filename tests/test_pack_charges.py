"""lw.pack_charges by columns against one record at a time, over the forms a caller's charges
take: column types, strides and orders, more rows than kinds, single columns as lists or
tensors; and what one way refuses the other refuses."""
import numpy as np
import pytest
import torch

from paper_2107_12437_amd import inputs as I
from paper_2107_12437_amd import lw


def by_records(charges, monkeypatch):
    with monkeypatch.context() as m:
        m.setattr(lw, "_pack_columns", lambda *a: None)
        return lw.pack_charges(charges)


FORMS = {
    "plain": lambda c: c,
    "float32": lambda c: {k: v.astype(np.float32) if k != "kind" else v for k, v in c.items()},
    "integers": lambda c: {k: (np.sign(v) * 3).astype(np.int16) if k != "kind" else v.astype(np.uint8)
                           for k, v in c.items()},
    "complex": lambda c: dict(c, amp=c["amp"] + 0j),
    "half and long": lambda c: dict(c, phase=c["phase"].astype(np.float16), amp=c["amp"].astype(np.longdouble)),
    "column order": lambda c: {k: np.asfortranarray(v) for k, v in c.items()},
    "reversed": lambda c: {k: v[::-1] for k, v in c.items()},
    "every second": lambda c: {k: np.repeat(v, 2, axis=0)[::2] for k, v in c.items()},
    "more rows": lambda c: {k: v if k == "kind" else np.concatenate([v, v]) for k, v in c.items()},
    "a list": lambda c: dict(c, q=[float(x) for x in c["q"]]),
    "lists": lambda c: {k: v.tolist() for k, v in c.items()},
    "tensors": lambda c: {k: torch.tensor(v) for k, v in c.items()},
    "float kinds": lambda c: dict(c, kind=c["kind"].astype(np.float64) + 0.3),
    "wide kinds": lambda c: dict(c, kind=c["kind"].astype(np.int64) + (1 << 32)),
    "special values": lambda c: dict(c, omega=np.where(np.arange(len(c["q"])) % 2, np.nan, np.inf),
                                     phase=-np.zeros(len(c["q"]))),
}


@pytest.mark.filterwarnings("ignore:Casting complex")
@pytest.mark.parametrize("n", [0, 1, 2, 3, 7, 300])
@pytest.mark.parametrize("form", FORMS)
def test_columns_equal_records(form, n, monkeypatch):
    c = FORMS[form](I.random_grid_charges(np.random.default_rng(n), n) if n else
                    {k: v[:0] for k, v in I.random_grid_charges(np.random.default_rng(1), 1).items()})
    got, ng = lw.pack_charges(c)
    ref, nr = by_records(c, monkeypatch)
    assert ng == nr == n and len(got) == len(ref) and bytes(got) == bytes(ref)


def short(c, key):
    return dict(c, **{key: c[key][:-1]})


@pytest.mark.parametrize("spoil", [
    lambda c: short(c, "q"), lambda c: short(c, "v"), lambda c: dict(c, c0=c["c0"][:, :2]),
    lambda c: dict(c, e1=c["e1"][:, :1]), lambda c: dict(c, v=np.concatenate([c["v"], c["v"]], axis=1)),
    lambda c: dict(c, c0=c["c0"][:, 0]), lambda c: dict(c, amp=c["c0"]),
    lambda c: dict(c, phase=np.array(["x"] * len(c["q"]))), lambda c: {k: v for k, v in c.items() if k != "accel"},
], ids=range(9))
def test_refusals_stay(spoil, monkeypatch):
    c = spoil(I.random_grid_charges(np.random.default_rng(3), 5))
    with pytest.raises(Exception) as a:
        lw.pack_charges(c)
    with pytest.raises(type(a.value)):
        by_records(c, monkeypatch)
