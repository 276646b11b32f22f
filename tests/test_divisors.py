"""The division that nearly every kernel finds its place by: host code, the same on the device."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="ROCm clang++ not found")
def test_division_by_a_product_and_a_shift(tmp_path):
    """All divisors up to 70000, those about the powers of two, and 200000 others of every length: numbers about multiples and about both ends are divided exactly, and nothing is
    shifted by more than a word has."""
    exe = str(tmp_path / "divisors")
    build = subprocess.run([CLANG, "-std=c++17", "-O1", "-g", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                            "-I" + os.path.join(ROOT, "paper_2604_28175_amd", "csrc"), os.path.join(ROOT, "tests", "native", "divisors.cpp"), "-o", exe],
                           capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "quotients" in run.stdout, run.stdout[-500:] + run.stderr[-1500:]
