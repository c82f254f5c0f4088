"""Generated gfx950 code of the FP64 slot kernel: the loads of a node's
populations are issued together, not in groups with waits between (which cost
the AA pull 5 to 9%).  Compiles that kernel alone with the library's flags."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1610_01388_amd import build

Q = {1: 19, 2: 27}


@pytest.mark.parametrize("lat", [1, 2])
def test_slot_pull_issues_its_loads_together(lat, tmp_path):
    if not (shutil.which(build.HIPCC) or os.path.exists(build.HIPCC)):
        pytest.skip("no hipcc")
    src, out = tmp_path / "one.hip", tmp_path / "one.s"
    src.write_text('#include "step_impl.hpp"\nnamespace lbm {\n' + "".join(
        f"template __global__ void k_pull_slots<{lat}, {op}, PREC_F64, PAT_AA_PULL, false>(StepArgs);\n"
        for op in ("OP_IR", "OP_PR")) + "}\n")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--offload-device-only", str(src), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    best = {}
    name, run = None, 0
    for line in out.read_text().splitlines():
        m = re.match(r"^(_ZN3lbm12k_pull_slots\S+):", line)
        if m:
            name, run = m.group(1), 0
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name:
            if re.match(r"^\s+global_load_dwordx2\b", line):
                run += 1
                best[name] = max(best.get(name, 0), run)
            elif line.startswith(".LBB") or re.match(r"^\s+s_waitcnt\b.*vmcnt", line) or re.match(r"^\s+v_\w*f64\b", line):
                run = 0
    assert len(best) == 2 and all(n >= Q[lat] for n in best.values()), best
