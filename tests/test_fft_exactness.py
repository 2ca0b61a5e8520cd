"""The exactness argument of csrc/fft.h on the CPU: external products by its
butterflies, with digits and keys at their ends, against exact integers and
words; the distance from the integer and the key transform's error against the
header's bounds."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_12761_amd", "csrc")
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_products_round_to_the_exact_integers(tmp_path):
    exe = str(tmp_path / "exactness")
    build = subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-Wall", "-Werror", "-Wno-unknown-pragmas",
                            "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(ROCM, "include"), "-I", CSRC, "-o", exe,
                            os.path.join(ROOT, "tests", "fft", "exactness_driver.cpp"),
                            os.path.join(CSRC, "fft_tables.cpp"), "-lquadmath"],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    print(run.stdout)
    assert run.returncode == 0 and "exactness OK" in run.stdout, run.stdout[-2000:]
