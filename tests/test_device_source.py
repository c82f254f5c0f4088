"""The device sources hold no instruction in inline assembly (an empty one, which
only hides a value's history from the optimiser, is fine).  gfx950 needs wait
states between dependent instructions of some kinds, for instance two between a
vector instruction that writes a scalar register (the reload of a spilled lane
mask) and a vector instruction that reads it.  The compiler places them for the
instructions that it knows, and not in front of inline assembly."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1610_01388_amd", "csrc")


def test_no_instruction_in_inline_assembly():
    found = []
    files = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.hpp")))
    assert len(files) > 20
    for f in files:
        text = re.sub(r"//[^\n]*", "", open(f).read())
        for m in re.finditer(r"\b(?:__)?asm(?:__)?\s*(?:volatile|__volatile__)?\s*\(\s*\"([^\"]*)\"\s*([:)])", text):
            if m.group(2) == ")" and text[: m.start()].rstrip().endswith(")"):
                continue  # the assembler name of a declared function
            if m.group(1).strip():
                found.append((os.path.basename(f), m.group(1)))
    assert not found, found
