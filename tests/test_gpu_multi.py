"""GPU tests of several time steps per launch (small AA domains, compact
layout, default kernel form): the states have to be those of the per-step
kernels bit for bit (the row-segment kernel, selected by hand), over whole
boxes in one block, tiles with halos on one, two or three axes, walls,
periodic axes narrower than the halo, solids, tiles reaching past the domain,
odd step counts, monitor records in between, graph replays and several
streams."""
import numpy as np
import pytest

from support import random_mask

pytestmark = pytest.mark.gpu

NU, SY, G = 0.1, 4e-5, (4e-6, -2e-6, 1e-6)
# lattice, dims, periodic: one block, spanned and haloed axes, remainders
SHAPES = [("D2Q9", (4, 64, 1), (1, 0, 1)), ("D2Q9", (1, 1, 1), (1, 1, 1)), ("D2Q9", (5, 1, 1), (1, 0, 1)),
          ("D2Q9", (37, 41, 1), (1, 1, 1)), ("D2Q9", (3, 301, 1), (0, 0, 1)), ("D2Q9", (127, 66, 1), (0, 1, 1)),
          ("D3Q19", (8, 8, 8), (1, 0, 1)), ("D3Q19", (31, 29, 4), (0, 0, 1)), ("D3Q19", (65, 63, 3), (0, 1, 0)),
          ("D3Q19", (22, 23, 21), (1, 0, 0)), ("D3Q27", (9, 7, 5), (1, 0, 1)), ("D3Q27", (33, 17, 4), (0, 0, 1)),
          ("D3Q27", (5, 97, 2), (1, 1, 1))]


def make(lat, dims, per, op, precision, mask=None, stream=None):
    from paper_1610_01388_amd import lbm
    g = G if dims[2] > 1 else G[:2] + (0.0,)
    d = lbm.Domain(lat, dims, per, op, NU, SY, m=1e4 if op in ("PR", "PRI") else 0.0, g=g, precision=precision,
                   hb_n=0.7, stream=stream)
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
def test_equal_to_single_steps(op, precision):
    for k, (lat, dims, per) in enumerate(SHAPES):
        N = int(np.prod(dims))
        for mask in (None, random_mask(N, 60 + k, 0.2)):
            if mask is not None and (N < 16 or mask.all()):
                continue
            print(f"multi: {lat} {dims} {per} {op} {precision} solids {mask is not None}", flush=True)
            ref = make(lat, dims, per, op, precision, mask)
            ref.set_pull_form("ROWS")
            d = make(lat, dims, per, op, precision, mask)
            for n in (2, 46, 1, 9, 30):  # from odd times, in lengths the launches do not divide
                ref.step(n)
                d.step(n)
                assert same(state(d, op), state(ref, op)), (lat, dims, n)
            assert d.time == ref.time == 88
            ref.close()
            d.close()


@pytest.mark.parametrize("lat,dims,per,solid", [("D2Q9", (16, 33, 1), (1, 0, 1), 0), ("D2Q9", (80, 70, 1), (1, 1, 1), 1),
                                                ("D3Q19", (41, 38, 4), (0, 0, 1), 0)])
def test_monitors_and_graphs(lat, dims, per, solid):
    mask = random_mask(int(np.prod(dims)), 9, 0.2) if solid else None
    runs = []
    for form, graph in (("ROWS", 0), ("AUTO", 0), ("AUTO", 20)):
        d = make(lat, dims, per, "PR", "FP64", mask)
        d.set_pull_form(form)
        d.set_graph_steps(graph)
        d.set_monitor_interval(10)
        got = []
        for n in (40, 7, 13, 60, 41):  # replays, eager steps and host reads in turn
            d.step(n)
            got += state(d, "PR")
            got += [np.array([[h["step"], h["umax"], h["mass"], h["unyielded"], h["du_max"]] for h in d.history()])]
        runs.append(got)
        d.close()
    for other in runs[1:]:
        assert len(other) == len(runs[0]) and same(runs[0], other)  # states and records


def test_streams():
    import torch
    ref = make("D3Q19", (48, 40, 4), (0, 0, 1), "IR", "FP32")
    ref.set_pull_form("ROWS")
    ref.step(200)
    want = state(ref, "IR")
    streams = [torch.cuda.Stream() for _ in range(3)]
    doms = [make("D3Q19", (48, 40, 4), (0, 0, 1), "IR", "FP32", stream=s) for s in streams]
    for _ in range(10):
        for d in doms:
            d.step(20)
    for d in doms:
        assert same(state(d, "IR"), want)


def test_selected_forms_keep_their_kernels_and_autotune_keeps_state():
    d = make("D2Q9", (60, 50, 1), (1, 0, 1), "IR", "FP64")
    ref = make("D2Q9", (60, 50, 1), (1, 0, 1), "IR", "FP64")
    ref.set_pull_form("ROWS")
    d.step(33)
    ref.step(33)
    before = state(d, "IR")
    d.autotune(6)
    assert d.time == 33 and same(state(d, "IR"), before)
    d.set_tile(64, 2, 1)
    d.step(31)
    ref.step(31)
    assert same(state(d, "IR"), state(ref, "IR"))
