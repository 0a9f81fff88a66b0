"""Registers of the lane kernels as the compiler allots them (gfx950)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2110_15425_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    if not os.path.exists(build.HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("regs") / "sim_lane.o")
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-Rpass-analysis=kernel-resource-usage", "--offload-device-only",
                        "-c", os.path.join(build.CSRC, "sim_lane.hip"), "-o", out], capture_output=True, text=True,
                       check=True)
    found, name = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
        m = re.search(r"remark: .*?(VGPRs Spill|VGPRs|Occupancy \[waves/SIMD\]): (\d+)", line)
        if m and name:
            found.setdefault(name, {})[m.group(1)] = int(m.group(2))
    assert found
    return found


def test_time_course_spills_nothing(kernels):
    tc = {k: v for k, v in kernels.items() if "sim_lane_kernel" in k and "Lb1ELi0ELi256E" in k}
    assert len(tc) == 4, sorted(kernels)
    for k, v in tc.items():
        assert v["VGPRs Spill"] == 0, (k, v)
