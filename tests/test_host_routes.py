"""Which candidate path batches and plans take by the context's and a tuned
scene's sorted_candidates, what fits and in which shape: the library's host code with a
stubbed runtime (tests/host_fuzz/routes_host.cpp), on the CPU."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = os.path.join(ROOT, "tests", "host_fuzz", "routes_host.cpp")
HIP_INC = "/opt/rocm/include"


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    if not shutil.which("g++") or not os.path.isdir(HIP_INC):
        pytest.skip("g++ or the HIP runtime headers are not available")
    out = str(tmp_path_factory.mktemp("routes") / "routes_host")
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-D__HIP_PLATFORM_AMD__", "-I", HIP_INC,
                    "-I", os.path.join(ROOT, "paper_1911_06001_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    "-fsanitize=address,undefined", "-fno-sanitize-recover=all", "-Wno-subobject-linkage", SRC, "-o", out],
                   check=True, capture_output=True, text=True, timeout=300)

    def run(*args, cut=True):
        p = subprocess.run([out, *map(str, args)], capture_output=True, text=True, timeout=60)
        assert p.returncode == 0, p.stdout + p.stderr
        return [line.split()[:2] if cut else line.split() for line in p.stdout.splitlines()]

    return run


@pytest.mark.parametrize("context,tuned,candidates,path", [
    (0, -1, 16, "one-by-one"), (0, -1, 17, "hierarchy"),      # not tuned: the context's
    (0, 64, 64, "one-by-one"), (0, 17, 17, "one-by-one"),     # tuned one by one
    (0, 1, 16, "one-by-one"), (0, 16, 17, "hierarchy"),       # tuned to the hierarchy
    (64, 1, 64, "one-by-one"), (1, 1, 2, "hierarchy"),
])
def test_candidate_path_of_several_jobs(routes, context, tuned, candidates, path):
    assert routes(context, tuned, candidates, 2) == [["batch", path], ["plan", path]]


def test_tables_without_hierarchies_fit(routes):
    """28 jobs of 64 candidates: with their hierarchies the tables pass the
    LDS, one by one they do not."""
    assert routes(0, 64, 64, 28) == [["batch", "one-by-one"], ["plan", "one-by-one"]]
    assert [r[1] for r in routes(0, -1, 64, 28)] == ["refused:", "refused:"]


@pytest.mark.parametrize("waves,blocks,shape", [
    (8, 3, "8x3"), (4, 5, "4x5"), (12, 2, "12x2"), (2, 7, "2x7"),   # fit as they are
    (4, 6, "8x3"), (4, 8, "8x3"), (16, 2, "12x2"), (8, 4, "8x3"),   # most of their waves in larger work-groups
    (1, 32, "8x3"), (6, 5, "6x4"),
])
def test_shape_that_keeps_most_waves(routes, waves, blocks, shape):
    """Ten jobs of ten candidates: 7,040 B of tables in each work-group of a CU."""
    assert [r[3] for r in routes(0, -1, 10, 10, waves, blocks, cut=False)] == [shape, shape]


def test_one_work_group_takes_what_fits(routes):
    """28 jobs of 64 candidates leave room for 8 waves, 31 for 6."""
    assert routes(64, -1, 64, 28, 16, 2, cut=False)[0][3] == "8x1"
    assert routes(64, -1, 64, 31, 8, 3, cut=False)[0][3] == "6x1"
