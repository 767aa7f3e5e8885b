"""Exchanges between the lanes of a wave through LDS: a wave barrier orders no
memory by itself, so each one in the sources stands between a release fence
(the writes before it) and an acquire fence (the reads after it).
"""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_1608_06721_amd", "csrc")


def test_wave_barriers_are_fenced():
    seen = 0
    for path in sorted(glob.glob(os.path.join(CSRC, "*"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        stmts = [s.strip() for s in re.split(r"[;{}]", text)]
        for k, s in enumerate(stmts):
            if "__builtin_amdgcn_wave_barrier" not in s:
                continue
            seen += 1
            before, after = stmts[k - 1], stmts[k + 1]
            where = "%s: %s / %s" % (os.path.basename(path), before, after)
            assert re.search(r"amdgcn_fence\(__ATOMIC_(RELEASE|ACQ_REL), *\"wavefront\"", before), where
            assert re.search(r"amdgcn_fence\(__ATOMIC_(ACQUIRE|ACQ_REL), *\"wavefront\"", after), where
    assert seen > 0
