"""The FP32 tiles' decisions (CPU): compiles tests/c/tile_tables.cpp against
the library's edge compiler and runs it."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_certain_pairs_lie_in_their_band(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    from paper_1204_6630_amd.build import CSRC, HOST_FLAGS
    exe = str(tmp_path / "tile_tables")
    subprocess.check_call([cxx, *HOST_FLAGS, "-I" + CSRC, os.path.join(ROOT, "tests", "c", "tile_tables.cpp"),
                           os.path.join(CSRC, "edges.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout) > 1000000
