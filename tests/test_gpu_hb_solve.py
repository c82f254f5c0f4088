"""GPU tests of the FP64 Herschel-Bulkley solve where its single-precision
start is at its limits: flow indices at the ends of the accepted range, and
stresses so small that the start leaves the float range (n = 0.2: the root
goes with the fifth power of the excess stress) or that the linear term
decides (n = 5).  The oracle brackets the same root by bisection.

Tolerance: the post-collision stress is a Lipschitz function of the moments
(the solve's derivative is at most 2), so two correct FP64 runs differ by
rounding alone: at most about 27 terms of 1e-16 per node and step, 11 steps,
below 1e-13."""
import numpy as np
import pytest

from support import random_mask, run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0.2, 0.35, 1.0, 2.5, 5.0])
@pytest.mark.parametrize("amp,sigma_y", [(1e-2, 5e-5), (1e-6, 0.0), (1e-9, 0.0)])
def test_irhb_solve_range(n, amp, sigma_y):
    dims = (37, 29, 1)
    mask = random_mask(int(np.prod(dims)), 77, 0.1)
    ref, got, _, _ = run_pair(0, dims, (1, 0, 1), "IRHB", 11, mask=mask, seed=5, nu_p=0.05, sigma_y=sigma_y,
                              g=(amp * 1e-3, 0.0, 0.0), amp=amp, hb_n=n, pull_form="ROWS")
    assert np.isfinite(got[1]).all()
    assert np.max(np.abs(got[1] - ref[1])) <= 1e-13
    assert np.max(np.abs(got[0] - ref[0])) <= 1e-13
