"""Planes per workgroup of default tiles (tests/default_chunks_check.cpp, linked to
the library)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_default_chunks(tmp_path):
    from paper_2106_11286_amd import build as B

    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc) or not os.path.exists(B.LIB):
        pytest.skip("needs hipcc and the built library")
    exe = str(tmp_path / "default_chunks_check")
    subprocess.check_call([hipcc, "-std=c++17", "-O1", "-I", B.INCLUDE, "-I", B.CSRC,
                           "--offload-arch=" + B.ARCH, "-o", exe,
                           os.path.join(ROOT, "tests", "default_chunks_check.cpp"),
                           "-L" + os.path.dirname(B.LIB), "-l:" + os.path.basename(B.LIB),
                           "-Wl,-rpath," + os.path.dirname(B.LIB)])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
