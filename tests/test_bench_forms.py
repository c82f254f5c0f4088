"""bench.py's record of the kernel of a form, no GPU: a domain whose steps share
launches is not reported as a row kernel at a share of the HBM peak."""
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench  # noqa: E402


class Dom:
    def __init__(self, steps, tile):
        self.plan = (steps, tile)

    def steps_per_launch(self):
        return self.plan

    def pull_form(self):
        return "ROWS"


def test_kernel_fields():
    one = bench.kernel_fields(Dom(1, (0, 0, 0)), 4000.0)
    assert one == {"neighbour_kernel": "ROWS", "steps_per_launch": 1, "hbm_frac": 4000.0 / bench.HBM_PEAK_GBS}
    several = bench.kernel_fields(Dom(4, (8, 8, 4)), 4000.0)
    assert several == {"neighbour_kernel": None, "steps_per_launch": 4, "launch_tile": [8, 8, 4], "hbm_frac": None}
