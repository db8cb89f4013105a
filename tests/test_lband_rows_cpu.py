"""The LDS-staged band kernel copies rows of the lattice only, whatever the tile's
height (tests/lband_rows_check.cpp, host arithmetic)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_staged_rows_lie_in_the_lattice(tmp_path):
    from paper_2106_11286_amd import build as B

    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    exe = str(tmp_path / "lband_rows_check")
    subprocess.check_call([cxx, "-std=c++17", "-O1", "-I", B.CSRC, "-o", exe,
                           os.path.join(ROOT, "tests", "lband_rows_check.cpp")])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
