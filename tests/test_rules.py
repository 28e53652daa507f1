"""Rules that choose launch shapes and kernels (csrc/trig_rules.hpp), built with
g++ and run on the CPU."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "native", "rules_test.cpp")
INC = os.path.join(ROOT, "paper_1810_11966_amd", "csrc")


def test_launch_rules(tmp_path):
    exe = tmp_path / "rules_test"
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", INC, SRC, "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "all checks passed" in out.stdout
