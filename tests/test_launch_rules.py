"""Rules that choose a launch from sizes alone, on the CPU.  A small program
built with the host compiler against the library's internal header prints
them."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM_INCLUDE = "/opt/rocm/include"

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(ROCM_INCLUDE),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def lines(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("host") / "launch_rules")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE,
                           os.path.join(ROOT, "tests", "host", "launch_rules.cpp"), "-o", exe])
    out = {}
    for line in subprocess.check_output([exe], text=True).splitlines():
        name, *rest = line.split()
        out.setdefault(name, []).append([int(x) for x in rest])
    return out


def test_few_short_walks_take_one_neighbour_per_lane(lines):
    # a part-filled device is bound by a step's chain, which a second
    # neighbour per lane lengthens; only larger batches take two
    for max_n, walks, lanes, neighbours in lines["group2"]:
        assert lanes * neighbours >= max_n
        assert neighbours == (2 if max_n == 32 and walks > 4096 else 1)
