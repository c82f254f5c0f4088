"""GPU tests of domains whose rows hold a few nodes only, so that the row
kernel's tiles (64 nodes wide) outnumber the monitor slots of the work buffer:
by default they step whatever the number of steps (several per launch, then
single ones), with the same states and monitor records as the dense layout."""
import numpy as np
import pytest

from support import random_mask

pytestmark = pytest.mark.gpu


def make(lat, dims, per, op, scheme, layout, mask):
    from paper_1610_01388_amd import lbm
    d = lbm.Domain(lat, dims, per, op, 0.1, 4e-5, m=1e4 if op == "PR" else 0.0,
                   g=(4e-6, -2e-6, 1e-6 if dims[2] > 1 else 0.0), scheme=scheme, layout=layout)
    if mask is not None:
        d.set_mask(mask)
    d.init(1.0, (0.01, 0.02, 0.0))
    d.set_monitor_interval(7)
    return d


@pytest.mark.parametrize("scheme", ["AA", "AB"])
@pytest.mark.parametrize("lat,dims,per", [("D2Q9", (1, 400, 1), (1, 0, 1)), ("D2Q9", (3, 2001, 1), (0, 1, 1)),
                                          ("D3Q19", (3, 53, 50), (1, 0, 1)), ("D3Q27", (5, 60, 61), (1, 1, 0))])
def test_narrow_rows(lat, dims, per, scheme):
    from paper_1610_01388_amd import lbm
    N = int(np.prod(dims))
    for op in ("IR", "PR"):
        for mask in (None, random_mask(N, 21, 0.2)):
            d = make(lat, dims, per, op, scheme, "COMPACT", mask)
            ref = make(lat, dims, per, op, scheme, "DENSE", mask)
            assert d.pull_form() == "SLOTS"
            for n in (9, 1, 20, 3):
                d.step(n)
                ref.step(n)
                assert np.array_equal(d.read_populations()[0], ref.read_populations()[0]), n
            hd, hr = d.history(), ref.history()
            assert [h["step"] for h in hd] == [h["step"] for h in hr] == [0, 7, 14, 21, 28]
            for a, b in zip(hd, hr):
                assert a["umax"] == b["umax"] and a["unyielded"] == b["unyielded"] and a["nonfinite"] == 0
            d.set_pull_form("ROWS")
            with pytest.raises(lbm.LbmError):
                d.step(1)
            assert d.time == 33
            d.close()
            ref.close()
