"""The step kernel's LDS layout (csrc/kl_lds.h) on the host, over many shapes
(tests/cpu/lds_layout.cpp).  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_lds_layout(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "lds_layout")
    subprocess.run([gxx, "-std=c++17", "-O2", "-DKL_HD=",
                    "-I", os.path.join(ROOT, "paper_2410_23668_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"),
                    "-o", exe, os.path.join(ROOT, "tests", "cpu", "lds_layout.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "lds layout OK" in r.stdout
