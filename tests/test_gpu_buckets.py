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


@pytest.mark.parametrize("key", ["i64", "f32"])
@pytest.mark.parametrize("kv", [False, True], ids=["keys", "kv"])
def test_time_of_crowded_leaves(key, kv):
    """Segments of 100003 keys of 1000 widely spaced values: every leaf has bins of
    many equal keys.  Over the time of random keys each leaf may cost what a tile
    sort of as many keys costs, measured on segments of one short tile, and a
    tenth more."""
    import torch

    import paper_2305_05245_amd as pss

    n, seg = 160 * 100_003, 100_003
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    if key == "i64":
        random = torch.randint(-2**63, 2**63 - 1, (n,), dtype=torch.int64, device="cuda", generator=g)
    else:
        random = torch.rand(n, dtype=torch.float32, device="cuda", generator=g)
    some = random[:1000].clone()
    crowded = some[torch.randint(0, 1000, (n,), device="cuda", generator=g)].contiguous()
    vals = torch.arange(n, dtype=torch.int32, device="cuda") if kv else None

    def seconds(keys, length):
        offs = torch.arange(0, n // length * length + 1, length, dtype=torch.int64, device="cuda")
        times = []
        for _ in range(9):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            out, vout = pss.segmented_sort(keys, offs, vals, key_type=key, tuning={}, max_seg_len=length)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return sorted(times)[4], out, vout

    announce("crowded leaves", key, "kv" if kv else "keys")
    tiles, base = seconds(random, 4096)[0], seconds(random, seg)[0]
    t, out, vout = seconds(crowded, seg)
    print(f"random {base * 1e3:.0f} us, crowded {t * 1e3:.0f} us, tile sorts {tiles * 1e3:.0f} us")
    want, at = torch.sort(crowded.view(-1, seg), dim=1, stable=True)
    assert torch.equal(out, want.view(-1))
    if kv:
        assert torch.equal(vout, torch.gather(vals.view(-1, seg), 1, at).view(-1))
    assert t < 1.1 * (base + tiles)


def test_time_of_a_segment_above_its_bound():
    """A segment longer than the bound on the length, and no longer than the bound's
    merge passes reach, takes as many buckets as it needs: it may cost half as much
    again as with the right bound (one level of at most 384 buckets, where the right
    bound takes two)."""
    import torch

    import paper_2305_05245_amd as pss

    n = 8192 << 10
    keys = torch.randint(-2**63, 2**63 - 1, (n,), dtype=torch.int64, device="cuda")
    offs = torch.tensor([0, n // 8, n // 8 + 1_500_000, n // 8 + 1_500_000], device="cuda")
    offs[3:] = n // 8 + 1_500_000
    want = torch.sort(keys[n // 8:n // 8 + 1_500_000]).values

    def seconds(bound):
        times = []
        for _ in range(9):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            out, _ = pss.segmented_sort(keys, offs, tuning={}, max_seg_len=bound)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        assert torch.equal(out[n // 8:n // 8 + 1_500_000], want)
        return sorted(times)[4]

    announce("segment above its bound")
    right, low = seconds(1_500_000), seconds(263_000)
    print(f"right bound {right * 1e3:.0f} us, too low {low * 1e3:.0f} us")
    assert low < 1.5 * right


@pytest.mark.parametrize("kv", [False, True], ids=["keys", "kv"])
def test_time_of_segments_without_a_bound(kv):
    """Without a bound on the length the plan has the levels that one array would
    take; segments that one level can cut do not pay for the others.  The launches
    of a level without nodes take a few microseconds: a tenth of these sorts."""
    import torch

    import paper_2305_05245_amd as pss

    n, seg = 50 * 300_007, 300_007
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    some = torch.randint(-2**63, 2**63 - 1, (1000,), dtype=torch.int64, device="cuda", generator=g)
    keys = some[torch.randint(0, 1000, (n,), device="cuda", generator=g)].contiguous()
    vals = torch.arange(n, dtype=torch.int32, device="cuda") if kv else None
    offs = torch.arange(0, n + 1, seg, dtype=torch.int64, device="cuda")
    want, at = torch.sort(keys.view(-1, seg), dim=1, stable=True)

    def seconds(**bound):
        times = []
        for _ in range(9):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            out, vout = pss.segmented_sort(keys, offs, vals, tuning={}, **bound)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        assert torch.equal(out, want.view(-1))
        if kv:
            assert torch.equal(vout, torch.gather(vals.view(-1, seg), 1, at).view(-1))
        return sorted(times)[4]

    announce("segments without a bound", "kv" if kv else "keys")
    exact, none = seconds(max_seg_len=seg), seconds()
    print(f"bound given {exact * 1e3:.0f} us, none {none * 1e3:.0f} us")
    assert none < 1.1 * exact
