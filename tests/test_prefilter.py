"""Host constants of the prefilters (csrc/trig_bounds.hpp), built with g++ and
run on the CPU: the bound of the batched form's scan on pairs that pass the
pair test and the binned form's cells, up to the largest binary32 (paper Sec.
3.2, step 2)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "native", "prefilter_test.cpp")
INC = os.path.join(ROOT, "paper_1810_11966_amd", "csrc")


def test_prefilter_bounds(tmp_path):
    exe = tmp_path / "prefilter_test"
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-I", INC, SRC, "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stdout + out.stderr
    assert "all checks passed" in out.stdout
