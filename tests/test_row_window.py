"""The range-query planner's window of row counts: no load overwrites a row
that another wave may still read on the same side of the barrier, and every
row read was loaded before the last barrier (on the CPU, by the kernel's own
rule and its order of barriers, reads and loads).  The rule of one batch
earlier, planted in the model, is found out."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2008_03518_amd", "csrc")


@pytest.fixture(scope="module")
def model(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("row_window") / "row_window")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", CSRC, os.path.join(ROOT, "tests", "host", "row_window.cpp"),
                    "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("planted", [0, 1])
def test_no_load_over_rows_being_read(model, planted):
    out = subprocess.run([model, str(planted)], capture_output=True, text=True, check=True).stdout.split()
    missing, overwritten, loads = map(int, out)
    assert missing == 0 and loads > 10000
    assert (overwritten > 0) == bool(planted)
