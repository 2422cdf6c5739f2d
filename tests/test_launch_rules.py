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


def test_memetic_wavefronts_have_children_to_walk(lines):
    for words, replicas, K, children, gens, waves in lines["memetic"]:
        assert 1 <= waves <= min(12, gens * children)
        crowded = replicas > (512 if words == 4 else 2048)
        assert waves <= (12 if replicas <= 256 else 4 if crowded else 8)
        if replicas <= 512:
            assert waves == min(12 if replicas <= 256 else 8, gens * children)
        elif children == 1:
            # small populations: nearly every child waits for the one before it
            assert waves <= (1 + K // 6 if crowded else 2 + K // 8)
        else:
            # a generation's children walk side by side
            assert waves >= min(children, gens * children, 4)
        if K == 100 and gens >= 12:
            assert waves == (12 if replicas <= 256 else 4 if crowded else 8)


def test_populations_of_a_full_device_are_drawn_once(lines):
    for classes, replicas, waves in lines["init"]:
        assert waves == (4 if replicas <= (4096 if classes & 4 else 1024) else 1)


def test_tuned_launch_serves_its_own_batch_sizes(tmp_path):
    # a launch tuned on few walks is not used by a batch whose default is another form, nor the
    # reverse; nor is it lost where the default does not depend on the number
    from paper_2504_00987_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2504_00987_amd import build
        build.build()
    exe = str(tmp_path / "tuned_launch")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE,
                           os.path.join(ROOT, "tests", "host", "tuned_launch.cpp"), _lib.LIB_PATH,
                           "-Wl,-rpath," + os.path.dirname(_lib.LIB_PATH),
                           "-Wl,-rpath,/opt/rocm/lib", "-L/opt/rocm/lib", "-lamdhip64", "-o", exe])
    for line in subprocess.check_output([exe], text=True).splitlines():
        n, tuned, walks, used, same_default = (int(x) for x in line.split()[1:])
        assert used == same_default, line
