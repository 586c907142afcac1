"""Registers of the column sweeps with both coefficient arrays, from the compiler's report.

Their rings are the largest; a register spilled inside the plane loop costs more than a smaller window,
so a 16-bit sweep of two or four steps with both arrays takes the widest workgroup that spills none.
"""

import os
import re
import subprocess

import pytest

from paper_2504_09118_amd import build


@pytest.mark.skipif(not os.path.exists(build.HIPCC), reason="no hipcc")
@pytest.mark.parametrize("unit", ["k_column_f16.hip", "k_column_comp.hip"])
def test_both_arrays_spill_nothing(unit, tmp_path):
    cmd = [build.HIPCC, *build.FLAGS, "-w", "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
           "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(build.CSRC, unit),
           "-o", str(tmp_path / "unit.o")]
    res = subprocess.run(cmd, capture_output=True, text=True)
    assert res.returncode == 0, res.stderr
    name, spills = None, {}
    for line in res.stderr.splitlines():
        if m := re.search(r"Function Name: (\S+)", line):
            name = m[1]
        elif m := re.search(r"VGPRs Spill: (\d+)", line):
            spills[name] = int(m[1])
    # k_column<S, steps, Ce array, Ch array, waves>
    both = {n: v for n, v in spills.items() if re.search(r"k_column.*Li[24]ELb1ELb1ELi\d+E", n)}
    assert len(both) >= 4
    assert all(v == 0 for v in both.values()), both
