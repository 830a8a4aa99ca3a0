"""The host's rules of the Fourier-moment routes (csrc/dev_fourier.hpp):
tests/host/fourier_rules_test.cpp, the host half of a HIP compile, run here."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host", "fourier_rules_test.cpp")


def test_fourier_rules(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    exe = str(tmp_path / "fourier_rules")
    cmd = [hipcc, "-std=c++17", "-O2", "-x", "hip", "--offload-host-only", "-Wno-unused-function",
           "-I", os.path.join(ROOT, "paper_1804_11174_amd", "csrc"), SRC, "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "fourier rules ok" in r.stdout
