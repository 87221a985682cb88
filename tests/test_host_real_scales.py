"""The real-weight exact solver started from potentials far larger than the
weights (tests/host/real_start_scales.cpp, no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1104_3830_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")


def test_started_solves_equal_the_plain_ones_at_every_scale(tmp_path):
    exe = tmp_path / "real_start_scales"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D_GLIBCXX_ASSERTIONS", f"-I{CSRC}",
                    os.path.join(ROOT, "tests", "host", "real_start_scales.cpp"),
                    os.path.join(CSRC, "sk_solver_real.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr[-2000:]
    assert out.stdout.split()[1] == "solved=960"
