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


def _with_library(name, tmp_path):
    """The lines a program linked with the library prints."""
    from paper_2504_00987_amd import _lib
    if not os.path.exists(_lib.LIB_PATH):
        from paper_2504_00987_amd import build
        build.build()
    exe = str(tmp_path / name)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", ROCM_INCLUDE,
                           os.path.join(ROOT, "tests", "host", name + ".cpp"), _lib.LIB_PATH,
                           "-Wl,-rpath," + os.path.dirname(_lib.LIB_PATH),
                           "-Wl,-rpath,/opt/rocm/lib", "-L/opt/rocm/lib", "-lamdhip64", "-o", exe])
    return subprocess.check_output([exe], text=True).splitlines()


def test_few_short_walks_take_one_neighbour_per_lane(lines):
    # a part-filled device is bound by a step's chain, which a second
    # neighbour per lane lengthens; only larger batches take two
    for max_n, walks, lanes, neighbours in lines["group2"]:
        assert lanes * neighbours >= max_n
        assert neighbours == (2 if max_n == 32 and walks > 4096 else 1)


def test_memetic_wavefronts_have_children_to_walk(lines):
    for words, replicas, K, children, gens, waves in lines["memetic"]:
        full = replicas > (1024 if words == 4 else 2048)
        assert 1 <= waves <= min(12, gens * children)
        crowded = replicas > (512 if words == 4 else 2048)
        assert waves <= (12 if replicas <= 256 else 4 if crowded else 8)
        if replicas <= 512:
            assert waves == min(12 if replicas <= 256 else 8, gens * children)
        elif children == 1:
            # small populations: nearly every child waits for the one before it
            assert waves <= (1 + K // 8 if full else 2 + K // 8)
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
    for line in _with_library("tuned_launch", tmp_path):
        n, tuned, walks, used, same_default = (int(x) for x in line.split()[1:])
        assert used == same_default, line


@pytest.mark.parametrize("lanes", [64, 32, 16])
def test_walk_launches(lines, lanes):
    # what labs_tabu_batch launches: every present class in exactly one launch, in processing order;
    # one launch of one walk per wavefront at most, whose first class names its longest walk
    wave, short, shortest = 0, 2, 4  # kinds: one walk per wavefront, N <= 32, N <= 16
    for mask in range(1 << 8):
        present = [c for c in range(8) if mask >> c & 1]
        launches = [x[2:] for x in lines["launch"] if x[:2] == [mask, lanes]]
        covered = [c for f, z, _, _ in launches for c in range(f, z + 1) if c in present]
        assert covered == present
        assert all(f in present and z in present and f <= z for f, z, _, _ in launches)
        waves = [x for x in launches if x[2] == wave]
        assert len(waves) <= 1 and waves == launches[:len(waves)]
        for f, z, _, max_n in waves:
            assert f == present[0] and max_n == (256, 193, 128, 97, 64, 49, 32, 16)[f]
            assert lanes == 64 or z <= 5  # N <= 32 has a launch of its own
        kinds = [x[2] for x in launches[len(waves):]]
        want = [] if lanes == 64 else [c for c in (6, 7) if c in present]
        if lanes == 32:
            assert kinds == ([short] if want else [])
        else:
            assert kinds == [short if c == 6 else shortest for c in want]


def test_server_tables_out_of_memory(tmp_path):
    # LABS_E_NOMEM, no server, a message
    assert _with_library("server_tables", tmp_path) == ["2 1 1"] * 2
