"""The choice among timed tile shapes (csrc/ils_tune.hpp): stable between
candidates that are as fast as each other, the fastest otherwise."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_pick_is_stable(tmp_path):
    exe = str(tmp_path / "tune")
    subprocess.run(["g++", "-O2", "-std=c++17", os.path.join(ROOT, "tests", "native", "tune_check.cpp"), "-o", exe],
                   check=True, capture_output=True)
    run = subprocess.run([exe], capture_output=True, text=True)
    assert run.returncode == 0 and run.stdout.strip() == "passed", run.stdout
