"""The rules by which the workgroups of a short context's row count themselves, in every order (CPU only): the program beside this
file goes through them with the header the kernels include."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


def test_every_order_of_the_workgroups_of_a_row(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if not cxx:
        pytest.skip("a C++ compiler is needed")
    exe = str(tmp_path / "short_count_model")
    r = subprocess.run([cxx, "-O2", "-std=c++17", os.path.join(HERE, "short_count_model.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "passed" in r.stdout, r.stdout + r.stderr
