"""The shares that workgroups take of a phase's work (csrc/kl_shares.h), on
the host (tests/cpu/shares.cpp).  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_shares(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "shares")
    subprocess.run([gxx, "-std=c++17", "-O2", "-DKL_HD=",
                    "-I", os.path.join(ROOT, "paper_2410_23668_amd", "csrc"),
                    "-o", exe, os.path.join(ROOT, "tests", "cpu", "shares.cpp")], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "shares OK" in r.stdout
