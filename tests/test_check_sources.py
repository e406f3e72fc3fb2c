"""What the checking build can see.  A residual block's shortcut is read by
plain loads, not through buffer descriptors, so each of them has to stand
under the check of the output's extent (bufcheck.h); read from the sources,
since every caller of the kernels passes whole tensors.  And the calls that
the checking build and the run-twice test make have to reach every form of the
matrix-core kernels, whatever the dispatch sends elsewhere."""
import glob
import os
import re

import check_cases

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


def test_check_cases_reach_every_form():
    need = {"fold wavek", "dfp wavek", "group wavek", "fold fcx", "dfp fcx", "fold split K", "dfp split K"}
    need |= {f"{form} {out}" for out in ("f32", "codes", "res") for form in (
        "fold rows", "dfp two sets", "group u8 two sets", "group u4 two sets")}
    need |= {f"{form} {out}" for out in ("f32", "codes") for form in (
        "fold u8 one step", "fold u8 more steps", "fold u4 more steps", "dfp u8 one step", "dfp u8 more steps",
        "group u8 two steps", "group u8 more steps", "group u4 one step", "group u4 two steps",
        "group u4 more steps")}
    need |= {"fold u8 one step res", "fold u8 more steps res", "fold u4 more steps res singly",
             "dfp u8 one step res ahead", "dfp u8 more steps res behind", "dfp u8 more steps res ahead",
             "group u8 two steps res ahead", "group u8 two steps res singly", "group u8 more steps res behind",
             "group u4 two steps res ahead", "group u4 one step res singly", "group u4 more steps res behind"}
    assert not need - check_cases.forms()
