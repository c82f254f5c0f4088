"""GPU tests of very large TRT magic numbers, up to the limit where the odd
parts are not relaxed at all (infinity is accepted), against the oracle.

Tolerance: 11 steps of at most 27 terms, each rounded at 1e-16 of values below
1 and passed on by a collision whose derivatives stay below 30: 1e-12."""
import numpy as np
import pytest

from support import random_mask, run_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lam", [1e6, 1e300, float("inf")])
@pytest.mark.parametrize("op", ["PR", "PRI"])
@pytest.mark.parametrize("lat,dims", [(0, (37, 29, 1)), (2, (19, 9, 7))])
def test_large_magic_number(lat, dims, op, lam):
    mask = random_mask(int(np.prod(dims)), 13, 0.1)
    ref, got, pref, pgot = run_pair(lat, dims, (1, 0, 1), op, 11, mask=mask, seed=3, lam=lam, pull_form="ROWS")
    assert np.isfinite(pgot[0]).all()
    assert np.max(np.abs(pgot[0] - pref[0])) <= 1e-12
    assert np.max(np.abs(got[1] - ref[1])) <= 1e-12
