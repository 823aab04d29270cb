"""Buckets that the samples of the distribution sort miss, and what they cost."""
import numpy as np
import pytest

from gpu_util import KEY_OF_DTYPE, announce, order_bits, to_device
from test_gpu_distribution import _sample_positions, random_keys

pytestmark = pytest.mark.gpu


def _seconds(keys, vals=None, reps=5):
    """Median time of one sort, and its outputs."""
    import torch

    import paper_2305_05245_amd as pss

    dk, dv = to_device(keys), None if vals is None else to_device(vals)
    times = []
    for _ in range(reps):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        out, vout = pss.sort(dk, dv, key_type=KEY_OF_DTYPE[keys.dtype])
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1e-3)
    return (sorted(times)[reps // 2], out.cpu().numpy().view(keys.dtype),
            None if vals is None else vout.cpu().numpy().view(np.uint32))


@pytest.mark.parametrize("kv", [False, True], ids=["keys", "kv"])
def test_time_of_missed_buckets(kv):
    """Every sample holds the same key, so that two buckets hold half of the
    array each.  Merging them by pairs takes log2(n / tile) sweeps, here 7 or 8,
    by all workgroups, of about the time of the whole sort of random keys (7
    launches); one workgroup alone took 300 times as long."""
    n = 1_500_000 if not kv else 750_000
    rng = np.random.default_rng(1)
    plain = random_keys(rng, np.uint64, n)
    vals = rng.permutation(n).astype(np.uint32) if kv else None
    keys = plain.copy()
    for s in (4096, 8192):
        keys[_sample_positions(n, s)] = np.uint64(1 << 63)
    announce("missed buckets", n, "kv" if kv else "keys")
    base = _seconds(plain, vals)[0]
    t, out, vout = _seconds(keys, vals)
    print(f"random {base * 1e6:.0f} us, missed {t * 1e6:.0f} us")
    perm = np.argsort(order_bits(keys), kind="stable")
    assert out.tobytes() == keys[perm].tobytes()
    if kv:
        assert np.array_equal(vout, vals[perm])
    assert t < 20 * base
