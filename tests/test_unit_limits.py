"""Numbers and sizes of work units at the largest catalogs (CPU): compiles
tests/c/unit_limits.cpp against the library's unit header and runs it."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_units_of_the_largest_requests(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    exe = str(tmp_path / "unit_limits")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-Wall", "-I" + os.path.join(ROOT, "paper_1204_6630_amd", "csrc"),
                           os.path.join(ROOT, "tests", "c", "unit_limits.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout) > 400
