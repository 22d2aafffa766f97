"""Host-side check of the range in which the kernels' FP64 division and square
root are exact, and of what they give outside it."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_fp64_range(tmp_path):
    exe = tmp_path / "fp64_range_check"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-mfma", "-ffp-contract=off", "-o", str(exe),
                           os.path.join(HERE, "native", "fp64_range_check.cpp")])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
