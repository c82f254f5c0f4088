"""GPU tests of the batch's work-item order: what is selected and what is in
effect, plain order where it is asked for on an arena that the caches hold, and
arenas just below and above the sizes where the default changes (200 MB: chunks
to plain order; 512 MiB: streamed local phase), bit for bit against the
single-domain runs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def cases_of(sides, lattice="D3Q27"):
    return [dict(lattice=lattice, dims=(s, s - k, s + k), periodic=(k & 1, 0, 1), op="PR" if k == 1 else "IR", nu_p=0.1,
                 sigma_y=2e-5 * (k + 1), m=1e4 if k == 1 else 0.0, g=(2e-6, 0.0, 4e-6)) for k, s in enumerate(sides)]


def single(c, precision, steps):
    from paper_1610_01388_amd import lbm
    d = lbm.Domain(c["lattice"], c["dims"], c["periodic"], c["op"], c["nu_p"], c["sigma_y"], m=c["m"], g=c["g"],
                   precision=precision)
    d.step(steps)
    P = d.read_populations()[0]
    d.close()
    return P


def test_selection_and_effect():
    from paper_1610_01388_amd import lbm
    cases = cases_of((20, 33, 27, 25), "D3Q19")
    want = [single(c, "FP64", 9) for c in cases]
    for policy in (0, 1, 2, 3):
        for order, effect in ((-1, 1), (0, 0), (1, 1)):
            b = lbm.Batch(cases, precision="FP64")
            b.set_graph_steps(4)
            assert b.order() == (-1, 1) and b.schedule() == (3, 0)
            b.set_schedule(policy, max(order, 0))
            if order < 0:
                b.set_order(-1)
            assert b.order() == (order, effect)
            assert b.schedule() == (policy, max(order, 0))
            b.step(9)
            for k in range(len(cases)):
                assert np.array_equal(b.read_populations(k)[0], want[k]), (policy, order, k)
            b.close()
    b = lbm.Batch(cases, precision="FP64")
    for bad in (-2, 2):
        with pytest.raises(lbm.LbmError):
            b.set_order(bad)
    b.autotune(4)
    assert b.order()[0] in (0, 1) and b.order()[0] == b.order()[1]
    b.close()


@pytest.mark.parametrize("side,mb,effect", [(85, 199, 1), (86, 206, 0), (118, 532, 0), (119, 546, 0)])
def test_sizes_where_the_default_changes(side, mb, effect):
    from paper_1610_01388_amd import lbm
    cases = cases_of((side, side, side))
    b = lbm.Batch(cases, precision="FP32")
    nodes = sum((int(np.prod(c["dims"])) + 63) // 64 * 64 for c in cases)
    assert abs(nodes * 27 * 4 / 1e6 - mb) < 1
    assert b.order() == (-1, effect)
    b.step(7)
    for k in range(3):
        assert np.array_equal(b.read_populations(k)[0], single(cases[k], "FP32", 7)), k
    b.close()
