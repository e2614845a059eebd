"""The setup refuses cell-lane tables in which a step takes a stack entry that the
step before it left into: the kernels read the top entry one step ahead."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from workloads import configs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1810_12742_amd", "csrc")


def test_entry_taken_in_the_step_after_it_was_left_is_refused(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe, inp = str(tmp_path / "driver"), str(tmp_path / "forest.bin")
    subprocess.run(["g++", "-O1", "-std=c++17", "-pthread", "-o", exe, os.path.join(ROOT, "tests", "cell_stack_driver.cpp"),
                    *(os.path.join(CSRC, f) for f in ("setup.cpp", "cells.cpp", "resident.cpp"))], check=True)
    f = configs.c2(24).forest
    with open(inp, "wb") as fh:
        np.array([f.n, f.ncells], dtype=np.int64).tofile(fh)
        f.parent.astype(np.int32).tofile(fh)
        f.cell_offsets.astype(np.int64).tofile(fh)
    r = subprocess.run([exe, inp], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
