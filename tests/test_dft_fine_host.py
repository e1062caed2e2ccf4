"""The register DFTs of the plans of single FP32 calls (paper_1605_02060_amd/csrc/dft.h): closer
to the exact transform than those with constants rounded to FP32 (tests/dft_fine_host_check.cpp).
No GPU needed."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_both_parts_of_the_constants_are_closer(tmp_path):
    exe = tmp_path / "dft_fine_host_check"
    cmd = [HIPCC, "-O2", "-std=c++17", "-ffp-contract=on", "-x", "hip", "--offload-arch=gfx950",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I", os.path.join(ROOT, "paper_1605_02060_amd", "csrc"),
           os.path.join(ROOT, "tests", "dft_fine_host_check.cpp"), "-o", str(exe)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    print(out.stdout)
    assert out.returncode == 0, out.stdout
