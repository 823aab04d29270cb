"""The library's kernels on the CPU: every source of the sort compiled with g++
against a stand-in for the HIP runtime (native/hip_emu) and run under the
address and undefined-behaviour sanitizers, with the waves of a workgroup and
the workgroups of a launch in several orders."""
from __future__ import annotations

import concurrent.futures as cf
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")
CSRC = os.path.join(ROOT, "paper_2305_05245_amd", "csrc")
SOURCES = ["pss_api.hip", "pss_kernels.hip", "pss_dist.hip", "pss_noalloc.hip"]

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    tree = tmp_path_factory.mktemp("kernels")
    src = tree / "pkg" / "csrc"
    src.mkdir(parents=True)
    shutil.copytree(os.path.join(ROOT, "include"), tree / "include")
    for f in os.listdir(CSRC):
        if f.endswith((".hpp", ".hip")):
            # (the one constraint of an empty asm that names a vector register)
            text = open(os.path.join(CSRC, f)).read().replace('"+v"', '"+r"')
            (src / f).write_text(text)
    flags = ["-std=c++17", "-O1", "-g", "-w", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]
    inc = ["-I", os.path.join(NATIVE, "hip_emu"), "-I", str(tree / "include")]

    def compile_one(path):
        obj = str(tree / (os.path.basename(path) + ".o"))
        r = subprocess.run(["g++", *flags, *inc, "-x", "c++", "-c", path, "-o", obj],
                           capture_output=True, text=True, timeout=600)
        assert r.returncode == 0, r.stderr
        return obj

    paths = [str(src / f) for f in SOURCES] + [os.path.join(NATIVE, "kernels_on_host.cpp")]
    with cf.ThreadPoolExecutor(max_workers=len(paths)) as ex:
        objs = list(ex.map(compile_one, paths))
    exe = str(tree / "kernels_on_host")
    r = subprocess.run(["g++", *flags, *objs, "-o", exe], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr
    return exe


def run(program, case, seed):
    r = subprocess.run([program, case, str(seed)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and "passed" in r.stdout, f"{case}, seed {seed}\n{r.stdout}\n{r.stderr}"


@pytest.mark.parametrize("seed", [0, 1, 2, 3])
def test_segment_left_out(program, seed):
    run(program, "segment_left_out", seed)


@pytest.mark.parametrize("seed", [0, 1])
def test_plan_bounds(program, seed):
    run(program, "plan_bounds", seed)


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_big_buckets(program, seed):
    run(program, "big_buckets", seed)


@pytest.mark.parametrize("case", ["crowded_leaves", "leaf_bins", "segment_routes"])
@pytest.mark.parametrize("seed", [0, 1])
def test_leaves_and_segments(program, case, seed):
    run(program, case, seed)


@pytest.mark.parametrize("seed", [0, 1])
def test_doubled_splitters(program, seed):
    run(program, "doubled_splitters", seed)
