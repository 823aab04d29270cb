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
