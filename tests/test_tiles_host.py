"""The kernels' tile arithmetic and launch shapes, built for the host and
checked over whole ranges of sizes.  CPU only."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2608_23429_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
@pytest.mark.parametrize("program", ["tiles", "shapes"])
def test_host_arithmetic(tmp_path, program):
    exe = os.path.join(tmp_path, program + "_check")
    subprocess.run(["g++", "-std=c++17", "-O2", "-D__HIP_PLATFORM_AMD__", "-I", CSRC,
                    "-I", os.path.join(os.path.dirname(HERE), "include"),
                    "-I", os.path.join(ROCM, "include"),
                    os.path.join(HERE, program + "_check.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert program + " ok" in r.stdout
