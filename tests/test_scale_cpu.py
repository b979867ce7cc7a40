"""The scale of the iterate and the penalty's constants (csrc/ils_scale.hpp),
over penalties of every width: eps and gamma take effect as given, to a
rounding, and the scale cancels out of the result."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_scale_and_penalty_constants(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "scale")
    subprocess.run([HIPCC, "-x", "hip", "-O2", "-std=c++17", "--offload-arch=gfx950",
                    os.path.join(ROOT, "tests", "native", "scale_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0 and run.stdout.strip() == "passed", run.stdout[:2000]
