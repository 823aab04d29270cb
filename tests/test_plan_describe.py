"""What pss_plan_describe says of the sort that runs, and what the host code does
without the distribution kernels (CPU only)."""
from __future__ import annotations

import os
import shutil
import subprocess

import pytest

from paper_2305_05245_amd import _lib

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
NATIVE = os.path.join(ROOT, "tests", "native")


@pytest.mark.parametrize("kt,vt,n,levels,gathered,sweeps", [
    ("i64", 0, 8192, 0, False, 1.0),             # one tile
    ("i64", 0, 8193, 1, False, 2.0),             # partition, leaves
    ("f32", 0, 39_999, 0, False, 2.0),           # tiles, one merge pass
    ("f32", 0, 40_000, 1, False, 2.0),
    ("i64", 0, 384 * 4096 + 1, 2, False, 3.5),   # count, scatter, partition, leaves
    ("u64", 1, 384 * 2048 + 1, 2, False, 3.5),
    ("i64", 0, 1 << 28, 2, True, 3.0),           # partition, gathered partition, leaves
    ("u64", 1, 1 << 27, 2, True, 3.0),
    ("u64", 1, 300_000_000, 3, True, 4.5),
    ("u32", 0, 600_000_000, 3, False, 5.0),
])
def test_plan_says_what_runs(kt, vt, n, levels, gathered, sweeps):
    p = _lib.plan(_lib.KEY_NAMES[kt], vt, n)
    assert (p["bucket_levels"], p["gathered"], p["sweeps"]) == (levels, gathered, sweeps)


def test_paper_plan_is_merged():
    p = _lib.plan(_lib.I32, 0, 1 << 20, 64, 64)
    assert p["bucket_levels"] == 0 and p["sweeps"] == p["hbm_passes"] == 3


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_without_the_distribution_kernels(tmp_path):
    """A program linked without pss_dist.hip plans the same sorts and is refused
    when it runs one."""
    tree = tmp_path / "pkg" / "csrc"
    tree.mkdir(parents=True)
    csrc = os.path.join(ROOT, "paper_2305_05245_amd", "csrc")
    for f in os.listdir(csrc):
        if f.endswith((".hpp", ".hip")):
            shutil.copy(os.path.join(csrc, f), tree / f)
    shutil.copytree(os.path.join(ROOT, "include"), tmp_path / "include")
    main = tmp_path / "main.cpp"
    main.write_text("""
#include <cstdio>
#include <cstring>
#include <vector>
#include "pss.h"
int main() {
  pss_ctx *c = nullptr;
  if (pss_create(0, &c) != PSS_OK) return 2;
  char buf[1024];
  if (pss_plan_describe(PSS_I64, PSS_VAL_NONE, 1 << 28, 0, 0, buf, sizeof buf) != PSS_OK) return 3;
  if (!std::strstr(buf, "\\"bucket_levels\\": 2")) return 4;
  std::vector<long long> k(10000), o(10000);
  std::vector<char> ws(1 << 20);
  if (pss_sort(c, PSS_I64, PSS_VAL_NONE, k.data(), o.data(), nullptr, nullptr, 10000, 0, 0, ws.data(),
               ws.size(), nullptr) != PSS_ERR_UNSUPPORTED) return 5;
  std::printf("%s\\n", pss_last_error(c));
  pss_destroy(c);
}
""")
    exe = str(tmp_path / "main")
    inc = ["-I", os.path.join(NATIVE, "hip_emu"), "-I", str(tmp_path / "include")]
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", *inc, "-x", "c++", str(tree / "pss_api.hip"),
                        os.path.join(NATIVE, "kernel_stubs.cpp"), str(main), "-o", exe],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "without pss_dist.hip" in r.stdout, (r.returncode, r.stdout, r.stderr)
