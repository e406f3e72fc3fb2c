"""What the checking build can see of a residual block's shortcut: it is read
by plain loads, not through buffer descriptors, so each of them has to stand
under the check of the output's extent (bufcheck.h).  Read from the sources,
since every caller of the kernels passes whole tensors."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
# a shortcut's pointer with an offset: res + e, a.res[e], out.res + e
LOAD = re.compile(r"\bres \+ |\.res\[")


def test_residual_loads_are_checked():
    found = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_1705_01462_amd", "csrc", "*.h*"))):
        lines = [l.split("//")[0].rstrip() for l in open(path)]
        for i, line in enumerate(lines):
            if LOAD.search(line):
                found += 1
                first = i if line.lstrip().startswith("if") or lines[i - 1].endswith(";") else i - 1
                assert "check_store(kSiteStoreY" in " ".join(lines[first:i + 1]), f"{path}:{i + 1}"
    assert found >= 5
