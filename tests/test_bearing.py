"""The run's square root and quotients (bearing.h) round as sqrt and / do, also
next to the middle between two doubles; the unrefined reciprocal, planted in
the model, does not (on the CPU)."""
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
    exe = str(tmp_path_factory.mktemp("bearing") / "bearing")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "bearing.cpp"), "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("planted", [0, 1])
def test_rounded_as_sqrt_and_division(model, planted):
    out = subprocess.run([model, str(planted)], capture_output=True, text=True, check=True).stdout.split()
    root, quot, hard, n_hard = map(int, out)
    print(out)
    assert n_hard > 100000 and root == 0 and quot == 0
    assert (hard > 0) == bool(planted)
