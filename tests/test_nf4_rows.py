"""The engine's NF4 quantizer looks codes up in the row table of csrc/nf4.hpp by
float arithmetic. Replayed on the host (nf4_row_check.cpp), every code equals
the number of the oracle's midpoints strictly below x."""
import os
import shutil
import subprocess

import numpy as np
import pytest


def test_row_table_is_the_nearest_value_rule(orc, tmp_path):
    from oracle import nf4
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    exe = tmp_path / "nf4_row_check"
    subprocess.run(["g++", "-std=c++17", "-O2", "-ffp-contract=off", "-march=x86-64-v3", "-pthread",
                    "-I" + os.path.join(root, "paper_2306_10015_amd", "csrc"),
                    os.path.join(root, "tests", "nf4_row_check.cpp"), "-o", str(exe)], check=True)
    mids = " ".join(f"{int(u):08x}" for u in nf4.midpoints().astype(np.float32).view(np.uint32))
    r = subprocess.run([str(exe)], input=mids, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert " 0 mismatches" in r.stdout
