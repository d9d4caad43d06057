"""The digits and masks of few-query scoring (fp6 x fp4) over their whole range, on the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_mask_digits_on_the_host(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    exe = str(tmp_path / "mask_digits")
    subprocess.run(["g++", "-O1", "-std=c++17", "-fsanitize=undefined", "-D__HIP_PLATFORM_AMD__=1", "-I/opt/rocm/include",
                    os.path.join(ROOT, "tests", "host", "mask_digits.cpp"), "-o", exe], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "digits ok" in r.stdout and r.stderr == "", r.stdout + r.stderr
