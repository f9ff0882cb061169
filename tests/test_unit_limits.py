"""Numbers and sizes of work units at the largest catalogs, and the walks over
their columns, and the order of unit lists (CPU): compiles unit_limits.cpp,
column_parts.cpp and unit_order.cpp of tests/c against the library's unit
header and runs them."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(name, tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no g++")
    exe = str(tmp_path / name)
    subprocess.check_call([cxx, "-O2", "-std=c++17", "-Wall", "-I" + os.path.join(ROOT, "paper_1204_6630_amd", "csrc"),
                           os.path.join(ROOT, "tests", "c", name + ".cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout
    return int(out.stdout)


def test_units_of_the_largest_requests(tmp_path):
    assert _run("unit_limits", tmp_path) > 400


def test_columns_up_to_the_last(tmp_path):
    assert _run("column_parts", tmp_path) > 70


def test_unit_lists_are_ordered_stably(tmp_path):
    assert _run("unit_order", tmp_path) == 54
