"""The rules of the density propagation's coarse form, on the host."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_coarse_form_fits_its_kernel(tmp_path):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "density_plan_check")
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-ffp-contract=off", "-w",
                    "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "helpers", "density_plan_check.hip"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
