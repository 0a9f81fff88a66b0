"""The double-precision Box-Muller pair of the simulation kernels, on the host."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# Relative error in units of 2^-53: rho 1.6 (its rounding, half of the rounding
# of -2 ln u and the square root's residual), the table's value 2 (its rounding,
# at most doubled by the angle sum), the angle sum's correction 3, its product
# with rho 1, the last sum 1.
BOUND = 8.6


def test_normals64_against_80_bit(tmp_path):
    if not os.path.exists(HIPCC) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "normal64_check")
    subprocess.run([HIPCC, "-O2", "-std=c++17", "-ffp-contract=off",
                    os.path.join(HERE, "helpers", "normal64_check.hip"), "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe, str(BOUND)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
