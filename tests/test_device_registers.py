"""Vector registers of the arithmetic-bound kernels in the built code object
(CPU only): with more than 256 one wave is left on each SIMD.
"""
import re
import subprocess

import pytest

from test_device_code import code_object, tool  # noqa: F401  (fixture)


@pytest.mark.parametrize("kernel", ["k_blu_half", "kb_blu_half", "k_assemble", "kb_assemble"])
def test_two_waves_per_simd(code_object, kernel):  # noqa: F811
    notes = subprocess.run([tool("llvm-readelf"), "--notes", code_object], check=True,
                           capture_output=True, text=True).stdout
    recs = re.findall(r"\.symbol:\s+(\S+).*?\.vgpr_count:\s+(\d+)", notes, re.S)
    mine = [(n, int(v)) for n, v in recs if re.search(r"\d%sI" % kernel, n)]
    # every flux, in 1D and 2D (HLLC in 2D only)
    assert len(mine) >= 5, mine
    assert max(v for _, v in mine) <= 256, [m for m in mine if m[1] > 256]
