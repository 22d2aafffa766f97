"""Host-side check of the rules by size that choose a call's way (the same
header the library uses) against measured times."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_rules_take_the_faster_way(tmp_path):
    exe = tmp_path / "rules_check"
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-o", str(exe), os.path.join(HERE, "native", "rules_check.cpp")])
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
