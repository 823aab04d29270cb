"""Which kernels sort what, from the launches the library records, and the routes
that only long arrays take: three levels of buckets, and three and four merge passes
inside the blocks of the paper's single level."""
import numpy as np
import pytest

from gpu_util import announce, gpu_sort, order_bits
from test_gpu_distribution import TILE, check, random_keys

pytestmark = pytest.mark.gpu


def _launches(call):
    """Launches per kernel family of one call, and its result."""
    import paper_2305_05245_amd as pss

    pss.profile(True)
    try:
        pss.profile_read()
        result = call()
        return {k: v["launches"] for k, v in pss.profile_read().items()}, result
    finally:
        pss.profile(False)


@pytest.mark.parametrize("dtype,n,buckets", [
    (np.int32, 8192, False), (np.int32, 8193, True), (np.uint64, 8192, False), (np.uint64, 8193, True),
    (np.float32, 39_999, False), (np.float32, 40_000, True), (np.float64, 39_999, False),
    (np.float64, 40_000, True)], ids=lambda x: x.__name__ if isinstance(x, type) else str(x))
@pytest.mark.parametrize("kv", [False, True], ids=["keys", "kv"])
def test_array_route(dtype, n, buckets, kv):
    rng = np.random.default_rng(n)
    keys = random_keys(rng, dtype, n)
    vals = np.arange(n, dtype=np.uint32) if kv else None
    announce("route", np.dtype(dtype).name, n, "kv" if kv else "keys")
    ran, (out, vout) = _launches(lambda: gpu_sort(keys, vals))
    assert ("dist_leaves" in ran) == buckets and ("tile_sort" in ran) != buckets
    perm = np.argsort(order_bits(keys), kind="stable")
    assert out.tobytes() == keys[perm].tobytes()
    if kv:
        assert np.array_equal(vout, perm.astype(np.uint32))


@pytest.mark.parametrize("sizes,bound,buckets", [
    ([100, 8192], 8192, False), ([100, 8193, 262_144], 262_144, False), ([100, 262_145], 262_145, True),
    ([100, 8193, 262_145], 0, False), ([262_145, 300_000, 262_144], 0, True)])
def test_segment_route(sizes, bound, buckets):
    """Segments of more than one merge pass's worth are distributed; without a
    bound on the length their mean decides."""
    import torch

    import paper_2305_05245_amd as pss

    keys = np.random.default_rng(1).integers(-2**62, 2**62, size=sum(sizes))
    offs = np.concatenate([[0], np.cumsum(sizes)])
    announce("segment route", sizes, bound)
    d_keys, d_offs = torch.from_numpy(keys).cuda(), torch.from_numpy(offs).cuda()
    ran, (out, _) = _launches(lambda: pss.segmented_sort(d_keys, d_offs, tuning={"max_seg_len": 0},
                                                         max_seg_len=bound or None))
    assert ("dist_leaves" in ran) == buckets and "tile_sort" in ran
    out = out.cpu().numpy()
    for lo, hi in zip(offs[:-1], offs[1:]):
        assert np.array_equal(out[lo:hi], np.sort(keys[lo:hi]))


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=lambda d: np.dtype(d).name)
@pytest.mark.parametrize("n", [40_000, 7 * TILE, 7 * TILE + 1, 8 * TILE - 1, 64 * TILE + 63, 100_003])
def test_float_sizes(dtype, n):
    """Floats that are distributed, at the edges of tiles: random bits, and normal
    ones with every special value among them."""
    rng = np.random.default_rng(n)
    normal = rng.standard_normal(n).astype(dtype)
    at = rng.integers(0, n, size=n // 20)
    normal[at] = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, -np.nan, 1e-40], dtype=dtype)[
        rng.integers(0, 7, size=at.size)]
    for keys in (random_keys(rng, dtype, n), normal):
        for kv in (False, True):
            announce("distributed floats", np.dtype(dtype).name, n, "kv" if kv else "keys")
            check(keys, kv)


def _sorted_as_torch(key, n, kv, kind, **blocks):
    import torch

    import paper_2305_05245_amd as pss

    dt = {"i32": torch.int32, "i64": torch.int64}[key]
    info = torch.iinfo(dt)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    keys = torch.randint(info.min, info.max, (n,), dtype=dt, device="cuda", generator=g)
    if kind == "half":  # one value makes up half of the keys: a bucket of every level
        keys[torch.rand(n, device="cuda", generator=g) < 0.5] = 12345
    vals = torch.arange(n, dtype=torch.int32, device="cuda") if kv else None
    ran, (out, vout) = _launches(lambda: pss.sort(keys, vals, key_type=key, **blocks))
    assert pss.device_check(0) == 0
    want = torch.sort(keys, stable=kv)
    assert torch.equal(out, want.values)
    if kv:
        assert torch.equal(vout, want.indices.to(torch.int32))
    return ran


@pytest.mark.parametrize("key,n,kv,gathered", [
    ("i32", 590_000_003, False, False), ("i64", 590_000_003, False, True), ("i64", 295_000_001, True, True), ("i32", 295_000_001, True, True)])
@pytest.mark.parametrize("kind", ["random", "half"])
def test_three_levels(key, n, kv, gathered, kind):
    """Three levels of buckets, whose last gathers its keys or, where its tables
    do not fit the workspace, follows a second level that scatters too."""
    from paper_2305_05245_amd import _lib

    plan = _lib.plan(_lib.KEY_NAMES[key], int(kv), n)
    assert plan["bucket_levels"] == 3 and plan["gathered"] == gathered
    announce("three levels", key, n, "kv" if kv else "keys", kind)
    ran = _sorted_as_torch(key, n, kv, kind)
    assert ran["dist_sample"] == 3 and ran["dist_scatter"] == (1 if gathered else 2)


@pytest.mark.parametrize("key,n,kv,passes", [
    ("i32", 18_000_001, False, 3), ("i32", 540_000_001, False, 4), ("i64", 33_000_001, True, 2),
    ("i64", 35_000_003, True, 3)])
def test_merge_passes_of_blocks(key, n, kv, passes):
    """The blocks of the paper's single level, two of them: several merge passes of
    32 runs, and with values two of 64 runs or three."""
    from paper_2305_05245_amd import _lib

    plan = _lib.plan(_lib.KEY_NAMES[key], int(kv), n, 2, 3)
    assert len(plan["block_passes"]) == passes
    if passes == 2:
        assert plan["block_passes"] == [64, 64]
    announce("merge passes of blocks", key, n, "kv" if kv else "keys", plan["block_passes"])
    ran = _sorted_as_torch(key, n, kv, "random", n_blocks=2, n_parts=3)
    assert ran["merge"] == passes
