"""The multigrid hierarchy's host code (amg.hpp) on the CPU, through
tests/host_multigrid.cpp built with g++."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_25403_amd", "csrc")
UNITS = ["mesh.cpp", "parts.cpp", "rules.cpp"]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")


def build(exe, flags):
    cmd = ["g++", "-std=c++17", "-fopenmp", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
           os.path.join(ROOT, "include"), "-I", CSRC] + flags
    cmd += [os.path.join(ROOT, "tests", "host_multigrid.cpp")]
    cmd += [os.path.join(CSRC, u) for u in UNITS] + ["-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    return build(str(tmp_path_factory.mktemp("mg") / "host_multigrid"), ["-O2"])


def run(exe, what, threads="4"):
    r = subprocess.run([exe, what], capture_output=True, text=True, timeout=600,
                       env=dict(os.environ, OMP_NUM_THREADS=threads))
    assert r.returncode == 0 and "ok" in r.stdout, (r.returncode, r.stdout[-2000:],
                                                    r.stderr[-4000:])
    return r.stdout


def test_the_last_product_fits_the_partial_sums_of_large_meshes(program):
    """1024^2 squares and 80^3 cubes are past 8192 blocks of the usual size."""
    run(program, "large")


def test_memory_that_runs_out_is_an_exception(program):
    """Also inside the parallel regions, where one that leaves ends the process."""
    run(program, "memory")


def test_too_many_entries_mean_no_hierarchy(program):
    """A product past the 32-bit row pointers is not read as an operand."""
    run(program, "entries")


def test_hierarchies_are_clean_under_sanitizers(tmp_path):
    """Both hierarchies of meshes of every kind under AddressSanitizer and
    UndefinedBehaviorSanitizer: indices in range, a symmetric positive cycle."""
    exe = build(str(tmp_path / "sanitized"),
                ["-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"])
    run(exe, "shapes")


def test_the_hierarchy_does_not_depend_on_the_threads(program):
    """Every bit of every product on one thread and on seven (the checks above
    without sanitizers)."""
    out = [run(program, "shapes", n) for n in ("1", "7")]
    assert out[0] == out[1] and out[0].count("rows") > 20


def test_launches_over_many_runs_keep_to_the_grid(program):
    """The shared launches of a batch take a run per y block, at most 65536."""
    run(program, "groups")
