"""Performance cases: the sorts a program asks of this package, by size, type and entry point.

A case is a dict of plain values.  `prepare` makes its inputs on the GPU from a
seed, `run` makes one pass through the public entry points, `exact` gives the
same outputs from torch alone and `work` the bytes one pass cannot do without.
Every sort here is exact, so outputs are compared bit for bit.
"""
from __future__ import annotations

import numpy as np
import torch

import paper_2305_05245_amd as pss
from paper_2305_05245_amd.segmented import SegmentedGraph

# torch holds unsigned keys in its signed types; the package is told the key type
_STORE = {"i32": torch.int32, "u32": torch.int32, "i64": torch.int64, "u64": torch.int64,
          "f32": torch.float32, "f64": torch.float64}
_WIDTH = {"i32": 4, "u32": 4, "f32": 4, "i64": 8, "u64": 8, "f64": 8}


def listed() -> list[dict]:
    return [
        # one short array: a call inside a larger program, all launches and latency
        {"name": "one array of 1000 i64", "kind": "sort", "key": "i64", "dist": "uniform",
         "values": False, "n": 1000},
        # a short ragged array of measurements with the index it came from (an argsort)
        {"name": "30011 f32 with index", "kind": "sort", "key": "f32", "dist": "normal",
         "values": True, "n": 30011},
        # a middling array whose length is no multiple of anything
        {"name": "1000003 i64", "kind": "sort", "key": "i64", "dist": "uniform", "values": False,
         "n": 1000003},
        # the paper's single level: 64 blocks, 64 partitions, the parity configuration
        {"name": "2^20 i32, 64 blocks", "kind": "level", "key": "i32", "dist": "uniform",
         "n": 1 << 20, "blocks": 64, "parts": 64},
        # the paper's UniformInt input at its larger size
        {"name": "10^8 u32", "kind": "sort", "key": "u32", "dist": "uniform", "values": False,
         "n": 10 ** 8},
        # column of reals, as a statistics or physics program sorts it
        {"name": "2^27 f64 normal", "kind": "sort", "key": "f64", "dist": "normal",
         "values": False, "n": 1 << 27},
        # the headline: the largest keys-only sort of the benchmark
        {"name": "2^28 i64", "kind": "sort", "key": "i64", "dist": "uniform", "values": False,
         "n": 1 << 28},
        # few distinct values: a column of categories
        {"name": "50000017 i64 mod 1000", "kind": "sort", "key": "i64", "dist": "mod1000",
         "values": False, "n": 50000017},
        # keys with their index, stable: the basis of argsort and of record sorts
        {"name": "2^27 u64 with index", "kind": "sort", "key": "u64", "dist": "uniform",
         "values": True, "n": 1 << 27},
        # many independent arrays of very different lengths in one call
        {"name": "4096 arrays of i64", "kind": "segmented", "key": "i64", "arrays": 4096,
         "lo_exp": 6.0, "hi_exp": 20.0},
        # a batch of queued requests, loaded and sorted through one captured graph
        {"name": "batch of 96 u64 requests", "kind": "batch", "key": "u64", "arrays": 96,
         "lo_exp": 10.0, "hi_exp": 20.0},
        # the paper's Particle records: 96 bytes sorted by their key
        {"name": "10^7 records of 96 bytes", "kind": "records", "key": "u64", "record_bytes": 96,
         "n": 10 ** 7},
    ]


def _size(rng, lo: float, hi: float) -> int:
    """Log-uniform, and mostly odd."""
    n = int(round(2.0 ** rng.uniform(lo, hi)))
    return n | 1 if rng.random() < 0.75 else n


def draw(rng) -> dict:
    kind = rng.choice(["sort"] * 6 + ["level", "segmented", "batch", "records"])
    if kind == "sort":
        values = rng.random() < 0.4
        key = rng.choice(sorted(_STORE))
        if key[0] == "f":
            dist = rng.choice(["normal", "unit"])
        else:
            dist = rng.choice(["uniform", "uniform", "mod1000", "swapped"])
        return {"kind": "sort", "key": key, "dist": dist, "values": values,
                "n": _size(rng, 8.0, 26.0 if values else 27.0)}
    if kind == "level":
        blocks = rng.choice([16, 48, 64, 100, 256])
        return {"kind": "level", "key": rng.choice(["i32", "i64", "f64"]), "dist": "uniform",
                "n": _size(rng, 18.0, 25.0), "blocks": blocks, "parts": blocks}
    if kind == "segmented":
        return {"kind": "segmented", "key": rng.choice(["i32", "i64", "f32"]),
                "arrays": int(2.0 ** rng.uniform(4.0, 12.0)), "lo_exp": 6.0,
                "hi_exp": round(rng.uniform(12.0, 19.0), 2)}
    if kind == "batch":
        return {"kind": "batch", "key": rng.choice(["u64", "i64"]), "arrays": rng.randint(8, 192),
                "lo_exp": 10.0, "hi_exp": round(rng.uniform(14.0, 20.0), 2)}
    return {"kind": "records", "key": "u64", "record_bytes": rng.choice([16, 32, 96]),
            "n": _size(rng, 16.0, 23.0)}


# ------------------------------------------------------------------- inputs
def _keys(key: str, dist: str, n: int, g: torch.Generator) -> torch.Tensor:
    dt = _STORE[key]
    if dist == "normal":
        return torch.randn(n, dtype=dt, device="cuda", generator=g)
    if dist == "unit" or (dist == "uniform" and dt.is_floating_point):
        return torch.rand(n, dtype=dt, device="cuda", generator=g)
    if dist == "mod1000":
        return torch.randint(0, 1000, (n,), dtype=dt, device="cuda", generator=g)
    if dist == "swapped":  # rising, with one position in a hundred moved
        k = torch.arange(n, dtype=dt, device="cuda").mul_(8)
        k += torch.randint(0, 8, (n,), dtype=dt, device="cuda", generator=g)
        m = max(n // 100, 2)
        at = torch.randint(0, n, (m,), device="cuda", generator=g).unique()
        k[at] = k[at[torch.randperm(at.numel(), device="cuda", generator=g)]]
        return k
    info = torch.iinfo(dt)
    # (the upper bound of randint is exclusive and has to fit the type)
    return torch.randint(info.min, info.max, (n,), dtype=dt, device="cuda", generator=g)


def _sizes(case: dict) -> np.ndarray:
    """Lengths of a batch's arrays, the same for every seed: a plan is made for them."""
    r = np.random.Generator(np.random.PCG64(12))
    u = r.uniform(case["lo_exp"], case["hi_exp"], size=case["arrays"])
    return np.rint(np.exp2(u)).astype(np.int64)


def prepare(case: dict, seed: int) -> dict:
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind, key = case["kind"], case["key"]
    s = {"kind": kind, "key": key}
    if kind in ("sort", "level"):
        n = case["n"]
        s["keys"] = _keys(key, case["dist"], n, g)
        s["vals"] = torch.arange(n, dtype=torch.int32, device="cuda") if case.get("values") else None
        s["blocks"], s["parts"] = case.get("blocks", 0), case.get("parts", 0)
    elif kind == "segmented":
        sizes = _sizes(case)
        offs = np.zeros(sizes.size + 1, dtype=np.int64)
        np.cumsum(sizes, out=offs[1:])
        s["keys"] = _keys(key, "uniform", int(offs[-1]), g)
        s["offsets"] = torch.from_numpy(offs).cuda()
        s["longest"] = int(sizes.max())
        s["out"] = torch.empty_like(s["keys"])
    elif kind == "batch":
        sizes = [int(x) for x in _sizes(case)]
        s["requests"] = [_keys(key, "uniform", n, g) for n in sizes]
        s["values"] = [torch.arange(n, dtype=torch.int32, device="cuda") for n in sizes]
        s["total"] = sum(sizes)
        # the resident buffers are sized above the batch, as a server sizes them
        s["graph"] = SegmentedGraph(s["total"] + s["total"] // 8, len(sizes) + 32, key, True,
                                    tuning={"max_seg_len": max(sizes)})
    else:
        words = case["record_bytes"] // 8
        s["records"] = _keys("i64", "uniform", case["n"] * words, g).view(torch.uint8).view(
            case["n"], case["record_bytes"])
    return s


# --------------------------------------------------------------------- pass
def run(s: dict):
    kind, key = s["kind"], s["key"]
    if kind in ("sort", "level"):
        out, vals = pss.sort(s["keys"], s["vals"], n_blocks=s["blocks"], n_parts=s["parts"],
                             key_type=key)
        return (out, vals) if vals is not None else out
    if kind == "segmented":
        out, _ = pss.segmented_sort(s["keys"], s["offsets"], key_type=key,
                                    max_seg_len=s["longest"], out=s["out"])
        return out
    if kind == "batch":
        graph, stream = s["graph"], torch.cuda.current_stream()
        graph.load(s["requests"], s["values"], stream)
        graph.run(stream)
        return graph.keys_out[:s["total"]], graph.vals_out[:s["total"]]
    return pss.sort_records(s["records"], key, key_offset=0)


def work(case: dict) -> dict:
    """Every input byte read once and every output byte written once."""
    kind = case["kind"]
    if kind == "records":
        return {"bytes": 2 * case["n"] * case["record_bytes"], "flops": 0}
    n = case["n"] if "n" in case else int(_sizes(case).sum())
    each = _WIDTH[case["key"]] + (4 if kind == "batch" or case.get("values") else 0)
    return {"bytes": 2 * n * each, "flops": 0}


# ---------------------------------------------------------------- reference
def _ordered(keys: torch.Tensor, key: str) -> torch.Tensor:
    """Keys torch sorts in the key type's order (no NaN and no -0.0 here)."""
    if key == "u64":
        return keys ^ torch.iinfo(torch.int64).min
    if key == "u32":
        return keys ^ torch.iinfo(torch.int32).min
    return keys


def _sorted(keys: torch.Tensor, vals, key: str):
    if vals is None:
        k = torch.sort(_ordered(keys, key)).values
        return _ordered(k, key)  # the map undoes itself
    at = torch.sort(_ordered(keys, key), stable=True).indices
    return keys[at], vals[at]


def exact(case: dict, seed: int):
    kind, key = case["kind"], case["key"]
    if kind == "batch":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        sizes = [int(x) for x in _sizes(case)]
        parts = [_keys(key, "uniform", n, g) for n in sizes]
        pairs = [_sorted(k, torch.arange(k.numel(), dtype=torch.int32, device="cuda"), key)
                 for k in parts]
        return torch.cat([p[0] for p in pairs]), torch.cat([p[1] for p in pairs])
    s = prepare(case, seed)
    if kind in ("sort", "level"):
        return _sorted(s["keys"], s["vals"], key)
    if kind == "segmented":
        o = s["offsets"].tolist()
        return torch.cat([_sorted(s["keys"][a:b], None, key) for a, b in zip(o[:-1], o[1:])])
    words = s["records"].view(torch.int64).view(case["n"], -1)
    at = torch.sort(_ordered(words[:, 0].contiguous(), key), stable=True).indices
    return s["records"][at]
