"""The transforms' twiddle tables on the CPU: one copy per process, whatever the
number of contexts and threads, and exact to 64 bits."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_12761_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_tables_are_made_once_and_exact(tmp_path):
    exe = str(tmp_path / "tables")
    build = subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-Werror", "-pthread", "-D__HIP_PLATFORM_AMD__",
                            "-I", os.path.join(ROCM, "include"), "-I", CSRC, "-o", exe,
                            os.path.join(ROOT, "tests", "fft", "tables_driver.cpp"),
                            os.path.join(CSRC, "fft_tables.cpp"), "-lquadmath"],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    print(run.stdout)
    assert run.returncode == 0 and "tables OK" in run.stdout, run.stdout
