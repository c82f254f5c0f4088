"""GPU tests of batches whose arena exceeds the caches (above 512 MB: the AA
local phase streams with non-temporal accesses and the items are walked in
plain order) and of one just below 400 MB (contiguous chunks per XCD): every
simulation checked bit for bit against its single-domain run, with a fused
monitor record on either phase."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,sides,op", [("FP32", (90, 97, 101, 90, 71, 96, 99, 93), "PR"),
                                                ("FP64", (90, 61, 97, 88), "IR"), ("FP64", (71, 65, 66), "PR")])
def test_large_arena(precision, sides, op):
    from paper_1610_01388_amd import lbm
    cases = [dict(lattice="D3Q27", dims=(s, s - 3, s + 2), periodic=(k & 1, 0, 1), op=op, nu_p=0.1, sigma_y=2e-5 * (k + 1),
                  m=1e4 if op == "PR" else 0.0, g=(2e-6, 0.0, 4e-6)) for k, s in enumerate(sides)]
    b = lbm.Batch(cases, precision=precision)
    b.set_monitor_interval(3)
    b.step(7)
    hist = b.history()
    assert len(hist) == 3
    for k in (0, len(sides) // 2, len(sides) - 1):
        c = cases[k]
        d = lbm.Domain(c["lattice"], c["dims"], c["periodic"], op, c["nu_p"], c["sigma_y"], m=c["m"], g=c["g"],
                       precision=precision)
        d.set_monitor_interval(3)
        d.step(7)
        P, tau = d.read_populations(with_tau=(op == "PR"))
        Pb, taub = b.read_populations(k, with_tau=(op == "PR"))
        assert np.array_equal(P, Pb) and (tau is None or np.array_equal(tau, taub))
        for rec, one in zip([h[k] for h in hist], d.history()):
            assert rec["umax"] == one["umax"] and rec["unyielded"] == one["unyielded"]
        d.close()
    b.close()
