"""The host side of the library when memory or a launch fails, on a pretended
device (tests/host/fake_api.hip, the CPU): a call that ends early leaves
nothing in flight that reads or writes the context's pinned memory, plans
arrive without the pinned buffer, the next call is not told of an error that
was dealt with, and a context needs no memory for the range query's index."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
E_DEVICE = -3


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if shutil.which(HIPCC) is None or shutil.which("g++") is None:
        pytest.skip("hipcc or g++ not available")
    d = str(tmp_path_factory.mktemp("fake_api"))
    csrc = os.path.join(ROOT, "paper_2008_03518_amd", "csrc")
    objs = []
    for src in (os.path.join(ROOT, "tests", "host", "fake_api.hip"), os.path.join(csrc, "api.hip")):
        objs.append(os.path.join(d, os.path.basename(src) + ".o"))
        subprocess.run([HIPCC, "--offload-arch=gfx950", "--offload-host-only", "-O1", "-w", "-std=c++17", "-I",
                        os.path.join(ROOT, "include"), "-I", csrc, "-c", src, "-o", objs[-1]], check=True)
    exe = os.path.join(d, "fake_api")
    # (the device code's image is the one symbol left out)
    subprocess.run(["g++", "-no-pie", *objs, "-Wl,--unresolved-symbols=ignore-in-object-files", "-lpthread", "-o", exe],
                   check=True)

    def run(*args):
        res = subprocess.run([exe, *map(str, args)], capture_output=True, text=True, timeout=60)
        assert res.returncode == 0, (args, res.returncode, res.stderr[-2000:])
        out = [dict((k, int(v)) for k, v in re.findall(r"(\w+)=(-?\d+)", l)) for l in res.stdout.splitlines()]
        print(args, out)
        return out

    return run


CALLS = [("request", 1), ("departures", 8), ("departures", 70), ("batch", 8), ("fcfs", 8)]


@pytest.mark.parametrize("call, n", CALLS)
def test_without_memory_for_the_buffer(fake, call, n):
    for fail in ("none", "no_host_memory"):
        first, second = fake(call, n, fail)
        assert first["rc"] == second["rc"] == 0 and first["whole"] == second["whole"] == 1
        assert first["pending"] == second["pending"] == 0


@pytest.mark.parametrize("call, n", CALLS)
def test_a_launch_that_fails(fake, call, n):
    first, second = fake(call, n, "no_gather")
    assert first["rc"] == E_DEVICE and first["pending"] == 0
    assert second["rc"] == 0 and second["whole"] == 1 and second["pending"] == 0


def test_without_memory_for_the_index(fake):
    """The context is made, and plans on the kernel that reads the table
    itself (one that needs the index would be refused by its launcher)."""
    for call in fake("no_index", 1):
        assert call["rc"] == 0 and call["whole"] == 1 and call["pending"] == 0
        assert call["range"] == 0 and call["other"] > 0
