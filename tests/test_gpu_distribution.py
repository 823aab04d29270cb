"""The distribution sort of the automatic plan (arrays longer than two tiles),
at the sizes and key distributions where its parts can go wrong, against
numpy's stable sort of the order bits (bit-exact, values included)."""
import numpy as np
import pytest

from gpu_util import announce, gpu_sort, order_bits

pytestmark = pytest.mark.gpu

TILE = 6144          # keys of a scatter or partition tile
TARGET, TARGET_KV = 4096, 2048
MAX_PICKS = 384      # more buckets than this take a second level


def check(keys, kv):
    vals = np.random.default_rng(keys.size).permutation(keys.size).astype(np.uint32) if kv else None
    got, vgot = gpu_sort(keys, vals)
    perm = np.argsort(order_bits(keys), kind="stable")
    assert got.tobytes() == keys[perm].tobytes()
    if kv:
        assert np.array_equal(vgot, vals[perm])


def random_keys(rng, dtype, n):
    size = np.dtype(dtype).itemsize
    return rng.integers(0, 256, size=n * size, dtype=np.uint8).view(dtype)


# the shortest array distributed, edges of tiles, ranges of several tiles, and
# both sides of the step from one level to two
SIZES = [16385, 3 * TILE, 3 * TILE + 1, 4 * TILE - 1, 64 * TILE + 63,
         MAX_PICKS * TARGET, MAX_PICKS * TARGET + 1, 2048 * TILE + 1]
SIZES_KV = SIZES[:5] + [MAX_PICKS * TARGET_KV, MAX_PICKS * TARGET_KV + 1, 2048 * TILE + 1]


@pytest.mark.parametrize("dtype", [np.uint32, np.int64, np.float64], ids=lambda d: np.dtype(d).name)
@pytest.mark.parametrize("i", range(len(SIZES)))
def test_sizes(dtype, i):
    for kv, n in ((False, SIZES[i]), (True, SIZES_KV[i])):
        announce("distribution", np.dtype(dtype).name, n, "kv" if kv else "keys")
        check(random_keys(np.random.default_rng(n), dtype, n), kv)


def _few(rng, n, dtype):       # 5 values, the type's lowest and highest among them
    v = np.array([0, 1, 2, 1000, np.iinfo(dtype).max], dtype=dtype)
    return v[rng.integers(0, 5, size=n)]


def _half(rng, n, dtype):      # one value makes up half of the keys
    k = random_keys(rng, dtype, n)
    k[rng.random(n) < 0.5] = 12345
    return k


def _copies(rng, n, dtype):    # about 40 copies of every value
    return rng.integers(0, max(n // 40, 1), size=n).astype(dtype)


def _powers(rng, n, dtype):    # spread over all magnitudes: crowded bins
    bits = np.iinfo(dtype).bits
    return (random_keys(rng, dtype, n) >> rng.integers(0, bits, size=n).astype(dtype)).astype(dtype)


def _sorted(rng, n, dtype):
    return np.sort(random_keys(rng, dtype, n))


def _reverse(rng, n, dtype):
    return np.sort(random_keys(rng, dtype, n))[::-1].copy()


def _period(rng, n, dtype):    # a ramp of 64 repeated
    return (np.arange(n) % 64).astype(dtype)


def _constant(rng, n, dtype):
    return np.full(n, np.iinfo(dtype).max, dtype=dtype)


@pytest.mark.parametrize("dtype", [np.uint32, np.uint64], ids=lambda d: np.dtype(d).name)
@pytest.mark.parametrize("make", [_few, _half, _copies, _powers, _sorted, _reverse, _period, _constant],
                         ids=lambda f: f.__name__[1:])
@pytest.mark.parametrize("n", [30011, 700_001, 3_000_017])
def test_distributions(n, make, dtype):
    keys = make(np.random.default_rng(n), n, dtype)
    for kv in (False, True):
        announce("distribution", make.__name__, np.dtype(dtype).name, n, "kv" if kv else "keys")
        check(keys, kv)


@pytest.mark.parametrize("dtype", [np.float32, np.float64], ids=lambda d: np.dtype(d).name)
@pytest.mark.parametrize("n", [30011, 2_500_003])
def test_float_specials(n, dtype):
    rng = np.random.default_rng(n)
    keys = rng.standard_normal(n).astype(dtype)
    at = rng.integers(0, n, size=n // 20)
    keys[at] = np.array([0.0, -0.0, np.inf, -np.inf, np.nan, -np.nan, 1e-40], dtype=dtype)[
        rng.integers(0, 7, size=at.size)]
    for kv in (False, True):
        announce("distribution floats", np.dtype(dtype).name, n, "kv" if kv else "keys")
        check(keys, kv)


def _sample_positions(n, samples):
    """Positions the first level samples: one hashed position in each of
    `samples` equal strata."""
    j = np.arange(samples, dtype=np.uint64)
    m = np.uint64(0xFFFFFFFF)
    h = (((j + np.uint64(1)) * np.uint64(0x9E3779B1)) & m) ^ np.uint64(0x85EBCA6B)
    h ^= h >> np.uint64(15)
    h = (h * np.uint64(0x2C1B3C6D)) & m
    h ^= h >> np.uint64(12)
    h = (h * np.uint64(0x297A2D39)) & m
    h ^= h >> np.uint64(15)
    return ((j * np.uint64(n) + ((h * np.uint64(n)) >> np.uint64(32))) // np.uint64(samples)).astype(np.int64)


@pytest.mark.parametrize("kv", [False, True], ids=["keys", "kv"])
@pytest.mark.parametrize("n,samples", [(50_001, (512, 1024, 2048)), (400_009, (4096, 8192)),
                                       (2_000_003, (1024, 2048, 4096))])
def test_buckets_the_samples_miss(n, samples, kv):
    """Every sampled position of the first level holds the same key, so that
    its two splitters leave buckets far larger than one workgroup sorts."""
    keys = random_keys(np.random.default_rng(n), np.uint64, n)
    for s in samples:
        keys[_sample_positions(n, s)] = np.uint64(1 << 63)
    announce("distribution, samples miss", n, "kv" if kv else "keys")
    check(keys, kv)


def _segmented(keys, sizes, vals=None, max_seg_len=None):
    """(sorted keys, sorted values, device error word) of one segmented sort
    on a poisoned workspace."""
    import torch

    import paper_2305_05245_amd as pss
    from gpu_util import KEY_OF_DTYPE, from_device, poisoned_workspace, to_device
    from paper_2305_05245_amd import _lib

    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    kt = _lib.KEY_NAMES[KEY_OF_DTYPE[keys.dtype]]
    vt = _lib.VAL_NONE if vals is None else _lib.VAL_U32
    tu = _lib.Tuning(2048, 4096, int(max_seg_len or max(sizes)), 0, 0)
    ws = poisoned_workspace(_lib.segmented_workspace_bytes(kt, vt, keys.size, len(sizes), tu))
    out, vout = pss.segmented_sort(to_device(keys), torch.from_numpy(offs).cuda(),
                                   None if vals is None else to_device(vals), key_type=kt, tuning=tu,
                                   workspace=ws)
    torch.cuda.synchronize()
    return (from_device(out, keys.dtype), None if vals is None else from_device(vout, np.uint32),
            pss.device_check(0), offs)


EDGES = [4096, 4097, 8192, 8193, 0, 3 * TILE, 3 * TILE + 1, 2048, 2049, 50_000, 1, 33 * 4096, 65 * TILE - 1]


@pytest.mark.parametrize("longest", [EDGES[-1], MAX_PICKS * TARGET, MAX_PICKS * TARGET + 1],
                         ids=["short", "one level", "two levels"])
@pytest.mark.parametrize("dtype", [np.uint32, np.int64], ids=lambda d: np.dtype(d).name)
def test_segments(dtype, longest):
    """Segments on both sides of every class: the two short ones, one leaf, a
    node of one tile and of several, nodes of few and of many buckets, and
    with a longer one in the batch the last single level and two levels."""
    sizes = EDGES + ([longest] if longest > max(EDGES) else [])
    rng = np.random.default_rng(longest)
    keys = random_keys(rng, dtype, sum(sizes))
    vals = rng.permutation(keys.size).astype(np.uint32)
    for v in (None, vals):
        announce("distribution segments", np.dtype(dtype).name, longest, "keys" if v is None else "kv")
        got, vgot, err, offs = _segmented(keys, sizes, v)
        assert err == 0
        for lo, hi in zip(offs[:-1], offs[1:]):
            perm = np.argsort(order_bits(keys[lo:hi]), kind="stable")
            assert got[lo:hi].tobytes() == keys[lo:hi][perm].tobytes()
            if v is not None:
                assert np.array_equal(vgot[lo:hi], vals[lo:hi][perm])


def test_segment_length_bound_too_small():
    """A bound on the segment length below the longest segment: up to the
    length that takes as many merge passes as the bound, the segment is sorted
    all the same; a longer one is left out and reported, the others are
    sorted."""
    rng = np.random.default_rng(3)
    for longest, reported in ((200_000, False), (32 * 8192 + 1, True)):
        sizes = [9000, longest, 100, 8200]
        keys = random_keys(rng, np.int64, sum(sizes))
        announce("distribution segments, bound 9000, longest", longest)
        got, _, err, offs = _segmented(keys, sizes, max_seg_len=9000)
        assert (err != 0) == reported and (err & 16 != 0) == reported
        for i, (lo, hi) in enumerate(zip(offs[:-1], offs[1:])):
            if not (reported and i == 1):
                assert np.array_equal(got[lo:hi], np.sort(keys[lo:hi]))


@pytest.mark.parametrize("copies", [2, 3, 6, 20, 96, 97, 255, 256])
@pytest.mark.parametrize("dtype", [np.uint32, np.int64], ids=lambda d: np.dtype(d).name)
def test_leaf_bins(dtype, copies):
    """One leaf of keys with several copies each: more bins to sort than the
    leaf's list holds at once (pairs), bins sorted in registers (3), by
    insertion (6), and up to the crowded limits.  Keys of all bits, and small
    ones whose bins hold one value each."""
    rng = np.random.default_rng(copies)
    for kv, n in ((False, 8192), (False, 8191), (True, 4096), (True, 4093)):
        for small in (False, True):
            each = random_keys(rng, dtype, n // copies + 1)
            if small:
                each = np.arange(each.size).astype(dtype)
            keys = rng.permutation(np.repeat(each, copies)[:n])
            vals = rng.permutation(n).astype(np.uint32) if kv else None
            announce("distribution leaf", np.dtype(dtype).name, copies, n, "kv" if kv else "keys")
            got, vgot, err, _ = _segmented(keys, [n], vals, max_seg_len=3 * TILE)
            assert err == 0
            perm = np.argsort(order_bits(keys), kind="stable")
            assert got.tobytes() == keys[perm].tobytes()
            if kv:
                assert np.array_equal(vgot, vals[perm])


@pytest.mark.parametrize("n", [1, 2, 63, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 8192])
def test_one_short_tile(n):
    """One array on both sides of each step of the workgroup that sorts it."""
    for dtype in (np.uint32, np.int64):
        for kv in (False, True):
            announce("one tile", np.dtype(dtype).name, n, "kv" if kv else "keys")
            keys = random_keys(np.random.default_rng(n), dtype, n)
            keys[: n // 3] = keys[-1]
            check(keys, kv)


GATHER_MIN = 1 << 25  # from here on the last of two levels gathers its keys


@pytest.mark.parametrize("kind", ["random", "sorted", "half", "copies", "powers", "runs"])
@pytest.mark.parametrize("dtype", ["int32", "int64"])
def test_gathered_level(dtype, kind):
    """The gathered last level against torch's stable sort: pieces of a few
    keys and of whole tiles, empty ones, and buckets that are not cut again
    (one value, or few keys)."""
    import torch

    import paper_2305_05245_amd as pss

    dt = getattr(torch, dtype)
    info = torch.iinfo(dt)
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    n = GATHER_MIN + 7 * TILE + 1
    keys = torch.randint(info.min, info.max, (n,), dtype=dt, device="cuda", generator=g)
    if kind == "sorted":
        keys = torch.sort(keys).values
    elif kind == "half":
        keys[torch.rand(n, device="cuda", generator=g) < 0.5] = 12345
    elif kind == "copies":
        keys = torch.randint(0, n // 40, (n,), dtype=dt, device="cuda", generator=g)
    elif kind == "powers":
        keys >>= torch.randint(0, info.bits, (n,), dtype=dt, device="cuda", generator=g)
    elif kind == "runs":    # sorted stretches, and a few low keys far apart
        m = n // 100_000
        keys[:m * 100_000] = torch.sort(keys[:m * 100_000].view(m, -1), dim=1).values.view(-1)
        keys[::50_021] = info.min
    want, at = torch.sort(keys, stable=True)
    vals = torch.randint(0, 1 << 31, (n,), dtype=torch.int64, device="cuda", generator=g).to(torch.int32)
    for v in (None, vals):
        announce("distribution, gathered", dtype, kind, n, "keys" if v is None else "kv")
        out, vout = pss.sort(keys, v, key_type="i32" if dtype == "int32" else "i64")
        assert torch.equal(out, want)
        if v is not None:
            assert torch.equal(vout, v[at])


@pytest.mark.parametrize("n", [8191, 8192, 8193, 8194, 39_999, 40_000])
@pytest.mark.parametrize("dtype", [np.int32, np.uint64, np.float32, np.float64],
                         ids=lambda d: np.dtype(d).name)
def test_shortest_distributed(dtype, n):
    """Both sides of the shortest arrays distributed, of random bits (floats:
    every special value), of 200 values (bins of one value) and normal ones."""
    rng = np.random.default_rng(n)
    few = rng.integers(0, 200, size=n)
    for keys in (random_keys(rng, dtype, n), few.astype(dtype),
                 (rng.standard_normal(n) * 1e6).astype(dtype)):
        for kv in (False, True):
            announce("shortest distributed", np.dtype(dtype).name, n, "kv" if kv else "keys")
            check(keys, kv)
