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


@pytest.mark.parametrize("block,waves", [(512, 2), (1024, 4)])
def test_default_bound_is_a_whole_number_of_workgroups(kernels, block, waves):
    """A workgroup of 512 or 1,024 threads puts 2 or 4 wavefronts on each SIMD: registers are
    not cut to a number of wavefronts that no number of workgroups makes up."""
    for mech, prec in (("DDM", 0), ("DDM", 1), ("LCA", 0), ("LCA", 1)):
        tag = f"{mech}ILi{prec}ELb0E"
        own = [v for k, v in kernels.items() if "sim_lane_kernel" in k and tag in k and f"Lb0ELi0ELi{block}E" in k]
        free = [v for k, v in kernels.items() if "sim_lane_kernel" in k and tag in k and f"Lb0ELi4ELi{block}E" in k]
        assert len(own) == 1 and len(free) == 1, tag
        # below four wavefronts' registers only where that holds another workgroup
        reach = own[0]["Occupancy [waves/SIMD]"] // waves * waves
        if reach <= 4:
            assert own[0]["VGPRs"] >= free[0]["VGPRs"] and own[0]["VGPRs Spill"] == 0, (tag, own, free)


def test_time_course_spills_nothing(kernels):
    tc = {k: v for k, v in kernels.items() if "sim_lane_kernel" in k and "Lb1ELi0ELi256E" in k}
    assert len(tc) == 4, sorted(kernels)
    for k, v in tc.items():
        assert v["VGPRs Spill"] == 0, (k, v)
