"""Coverage of the computed work units (CPU): compiles tests/c/unit_grid.cpp
against the library's unit header and runs it."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_pair_lies_in_one_unit(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    exe = str(tmp_path / "unit_grid")
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-Wall", "-I" + os.path.join(ROOT, "paper_1204_6630_amd", "csrc"),
                           os.path.join(ROOT, "tests", "c", "unit_grid.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout) > 800
