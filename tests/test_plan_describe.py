"""What pss_plan_describe says of the sort that runs (CPU only)."""
from __future__ import annotations

import pytest

from paper_2305_05245_amd import _lib


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
