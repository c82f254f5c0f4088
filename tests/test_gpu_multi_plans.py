"""GPU tests of several steps per launch where the caller selects the tile and
the steps: every operator and precision over boxes with halos on one, two and
three axes, more nodes than a block has threads, whole domains in one block,
solids, walls and periodic axes, bit for bit against single steps.  Each run
asserts that the selection is in effect."""
import numpy as np
import pytest

from support import random_mask

pytestmark = pytest.mark.gpu

# lattice, dims, periodic, tile, steps
PLANS = [("D2Q9", (13, 17, 1), (1, 0, 1), (0, 0, 0), 6),       # whole domain, one block
         ("D3Q27", (9, 7, 5), (0, 1, 1), (0, 0, 0), 4096),
         ("D2Q9", (40, 90, 1), (0, 1, 1), (0, 20, 0), 4),      # one cut axis, 1120 nodes in the box
         ("D2Q9", (47, 61, 1), (1, 0, 1), (10, 12, 0), 8),     # two, tiles past the domain
         ("D3Q19", (31, 29, 4), (0, 0, 1), (6, 7, 0), 4),
         ("D3Q19", (22, 23, 21), (1, 0, 0), (5, 5, 6), 2),     # three, 810 nodes
         ("D3Q27", (17, 13, 11), (0, 1, 1), (4, 4, 4), 2),
         ("D3Q27", (3, 2, 14), (1, 1, 0), (2, 1, 5), 2)]       # axes narrower than the halo


def make(lat, dims, per, op, precision, mask, **kw):
    from paper_1610_01388_amd import lbm
    g = (4e-6, -2e-6, 1e-6 if dims[2] > 1 else 0.0)
    d = lbm.Domain(lat, dims, per, op, 0.1, 4e-5, m=1e4 if op in ("PR", "PRI") else 0.0, g=g, precision=precision,
                   hb_n=0.7, **kw)
    if mask is not None:
        d.set_mask(mask)
    d.init(1.0, (0.02, -0.01, 0.005 if dims[2] > 1 else 0.0))
    return d


def state(d, op):
    P, tau = d.read_populations(with_tau=(op == "PR"))
    return [P] if tau is None else [P, tau]


def same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("precision", ["FP64", "FP32", "FP16"])
@pytest.mark.parametrize("op", ["IR", "PR", "PRI", "IRHB"])
@pytest.mark.parametrize("plan", range(len(PLANS)))
def test_selected_plans(plan, op, precision):
    lat, dims, per, tile, steps = PLANS[plan]
    for mask in (None, random_mask(int(np.prod(dims)), 80 + plan, 0.2)):
        print(f"plan: {PLANS[plan]} {op} {precision} solids {mask is not None}", flush=True)
        ref = make(lat, dims, per, op, precision, mask)
        ref.set_steps_per_launch(1)
        assert ref.steps_per_launch() == (1, (0, 0, 0))
        d = make(lat, dims, per, op, precision, mask)
        d.set_steps_per_launch(steps, tile)
        want = tuple(c if c else n for c, n in zip(tile, dims))
        for n in (2 * steps + 4 if steps < 100 else 12, 1, 9):
            assert d.steps_per_launch() == (steps, want)
            ref.step(n)
            d.step(n)
            assert same(state(d, op), state(ref, op)), n
        ref.close()
        d.close()


def test_chosen_where_it_pays():
    """Small domains, as used alone, take several steps by default."""
    for lat, dims, per, op, precision in (("D2Q9", (4, 64, 1), (1, 0, 1), "IR", "FP64"),
                                          ("D2Q9", (80, 80, 1), (1, 1, 1), "PR", "FP64"),
                                          ("D3Q19", (128, 128, 4), (0, 0, 1), "IR", "FP64"),
                                          ("D3Q27", (63, 63, 4), (0, 0, 1), "PR", "FP32")):
        d = make(lat, dims, per, op, precision, None)
        steps, tile = d.steps_per_launch()
        assert steps > 1 and all(1 <= c <= n for c, n in zip(tile, dims)), (lat, dims)
        for k, several in ((4, False), (5, True), (0, True)):
            d.set_monitor_interval(k)
            assert (d.steps_per_launch()[0] > 1) == several
        d.set_pull_form("ROWS")
        assert d.steps_per_launch() == (1, (0, 0, 0))
        d.set_pull_form("AUTO")
        d.set_steps_per_launch(1)
        assert d.steps_per_launch() == (1, (0, 0, 0))
        d.set_steps_per_launch(0)
        assert d.steps_per_launch() == (steps, tile)
        d.close()


def test_refused_selections():
    from paper_1610_01388_amd import lbm
    d = make("D3Q19", (40, 30, 20), (1, 0, 1), "IR", "FP64", None)
    for steps, tile in ((3, (8, 8, 4)), (-2, (8, 8, 4)), (4098, (8, 8, 4)), (4, (41, 8, 4)), (4, (8, -1, 4)),
                        (16, (8, 8, 4)), (2, (0, 0, 0))):
        with pytest.raises(lbm.LbmError):
            d.set_steps_per_launch(steps, tile)
    d.close()
    for kw in (dict(scheme="AB"), dict(layout="DENSE"), dict(mrt_even=1.2), dict(precision="FP32", fp64_fallback=True)):
        precision = kw.pop("precision", "FP64")
        d = make("D2Q9", (40, 30, 1), (1, 0, 1), "PR", precision, None, **kw)
        assert d.steps_per_launch() == (1, (0, 0, 0))
        with pytest.raises(lbm.LbmError):
            d.set_steps_per_launch(4, (8, 8, 0))
        d.close()


def test_selection_that_a_mask_makes_too_large():
    """6435 nodes a box: 148 KB without solids, 174 KB with them."""
    dims, per = (200, 150, 1), (1, 0, 1)
    d = make("D2Q9", dims, per, "IR", "FP16", None)
    ref = make("D2Q9", dims, per, "IR", "FP16", None)
    ref.set_steps_per_launch(1)
    d.set_steps_per_launch(2, (61, 95, 0))
    for mask in (None, random_mask(30000, 5, 0.1), np.zeros(30000, dtype=np.uint8)):
        for x in (d, ref):
            if mask is not None:
                x.set_mask(mask)
                x.init(1.0, (0.02, -0.01, 0.0))
            x.step(21)
        assert (d.steps_per_launch() == (2, (61, 95, 1))) == (mask is None or not mask.any())
        assert same(state(d, "IR"), state(ref, "IR"))


def test_default_walk_can_be_set_again():
    """Several steps per launch go with the default tile and order: another one
    turns them off, the default (by its values, or 0 for the order) on again."""
    d = make("D3Q19", (128, 128, 4), (0, 0, 1), "IR", "FP64", None)
    plan, tile, order = d.steps_per_launch(), d.tile(), d.tile_order()
    assert plan[0] > 1
    d.set_tile(*tile)
    d.set_tile_order(*order)
    assert d.steps_per_launch() == plan
    d.set_tile(64, 2, 1)
    assert d.steps_per_launch()[0] == 1
    d.set_tile(*tile)
    assert d.steps_per_launch() == plan
    d.set_tile_order(1, 1)
    assert d.steps_per_launch()[0] == 1
    d.set_tile_order(0, 0)
    assert d.steps_per_launch() == plan


def test_autotune_times_what_will_run():
    """Monitor intervals up to 4 leave single steps only, so a single-step form
    is tuned there; else several steps are timed in whole launches whatever the
    trial's length, and win on small domains."""
    for lat, dims, per, op in (("D2Q9", (80, 80, 1), (1, 1, 1), "PR"), ("D2Q9", (4, 64, 1), (1, 0, 1), "IR"),
                               ("D2Q9", (150, 150, 1), (1, 0, 1), "IR")):
        d = make(lat, dims, per, op, "FP64", None)
        plan = d.steps_per_launch()
        assert plan[0] > 1
        d.step(3)
        before = state(d, op)
        for interval, trial in ((0, 1), (0, 10), (7, 10), (40, 10), (100000, 3)):
            d.set_monitor_interval(interval)
            d.autotune(trial)
            assert d.steps_per_launch() == plan, (dims, interval, trial)
            assert d.time == 3 and same(state(d, op), before)
        d.set_monitor_interval(3)
        d.autotune(10)
        assert d.time == 3 and same(state(d, op), before)
        d.set_monitor_interval(0)
        assert d.steps_per_launch()[0] == 1
        d.close()


def test_autotune_drops_a_slow_selection():
    d = make("D3Q27", (60, 40, 24), (1, 0, 1), "IR", "FP64", None)
    d.set_steps_per_launch(2, (1, 1, 1))  # 125 nodes updated for one
    d.autotune(10)
    assert d.steps_per_launch()[0] == 1
    d.close()


@pytest.mark.parametrize("lat,dims,op,precision,solids", [
    ("D3Q19", (17, 19, 34), "IR", "FP16", 0.1),     # several / single 1.35
    ("D2Q9", (500, 500, 1), "IRHB", "FP64", 0.3),   # 1.19
    ("D2Q9", (500, 500, 1), "PRI", "FP64", 0.3),    # 1.17
    ("D2Q9", (700, 700, 1), "PR", "FP64", 0.3),     # 1.14
    ("D2Q9", (800, 800, 1), "IR", "FP64", 0.3)])    # 1.12
def test_single_steps_where_several_measured_slower(lat, dims, op, precision, solids):
    N = int(np.prod(dims))
    d = make(lat, dims, (1, 0, 1) if lat == "D2Q9" else (0, 0, 1), op, precision,
             random_mask(N, 5, solids) if solids else None)
    assert d.steps_per_launch()[0] == 1
    d.close()
