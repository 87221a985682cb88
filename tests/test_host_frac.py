"""The split of a logarithm into integer and fraction (sk_frac.h), built for
the host (tests/host/frac_check.cpp, no GPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1104_3830_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")


def test_a_split_logarithm_is_read_as_it_was_formed(tmp_path):
    exe = tmp_path / "frac_check"
    # HIP's own headers as system headers, without its device compiler
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-D__HIP_PLATFORM_AMD__", f"-I{CSRC}",
                    "-isystem", os.path.join(ROCM, "include"),
                    os.path.join(ROOT, "tests", "host", "frac_check.cpp"), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout[-2000:] + out.stderr[-2000:]
