"""The index arithmetic of the matrix-core GEMM (csrc/gemm_tiles.h), walked through on the host: no GPU needed."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not found")
def test_gemm_index_arithmetic_on_the_host(tmp_path):
    exe = str(tmp_path / "host_gemm_tiles_driver")
    r = subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", "-Wno-unused-command-line-argument",
                        "-I", os.path.join(ROOT, "paper_2412_01034_amd", "csrc"),
                        os.path.join(ROOT, "tests", "host_gemm_tiles_driver.cpp"), "-o", exe],
                       stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-4000:]
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and "gemm tiles: ok" in r.stdout, r.stdout[-4000:]
