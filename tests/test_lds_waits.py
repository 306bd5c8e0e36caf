"""Tiles that are loaded straight into LDS are published by full waits only.

The loads' order of completion in LDS is not relied on anywhere (a partial wait once let
the backward read a tile before all of it had landed), and a kernel that reads a tile too
early gives wrong values only now and then, so the rule is checked in the sources."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2609_38832_amd", "csrc")


def _code(path):
    return re.sub(r"//[^\n]*", "", open(path).read())


def test_only_full_vmcnt_waits():
    files = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h")))
    assert files
    seen = 0
    for f in files:
        code = _code(f)
        waits = re.findall(r"vmcnt\(([^)]*)\)", code) + re.findall(r"wait_vmcnt<([^>]*)>\(\);", code)
        waits = [w for w in waits if w.strip()]      # (the definition's own empty list)
        assert all(w.strip() == "0" for w in waits), (os.path.basename(f), waits)
        seen += len(waits)
    assert seen >= 4
