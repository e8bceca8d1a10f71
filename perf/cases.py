"""Performance cases: the sorts a program asks of this library, through the
Python binding's entry points, from a call of a thousand keys to 2^26.

A case is one call on one set of inputs: ``op`` names the entry point, ``n``
(or the segment table's recipe) the size, ``type`` the key type, ``kind`` the
distribution of the keys (the names of workloads.KINDS), ``ascending`` the
direction.  Sorting is in place, so a pass first copies the input into the
buffer it sorts, as a program does that keeps its input; the pass's outputs
are that buffer (and the values' buffer of a pair sort).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1506_01446_amd import binding as B
from paper_1506_01446_amd import workloads as W

ELEM = {"int32": 4, "uint32": 4, "float32": 4, "int64": 8, "uint64": 8, "float64": 8}

# Largest sizes drawn: a drawn case costs no more than the 2^26-key sort.
MAX_KEYS32 = 1 << 26
MAX_WIDE = 1 << 24
MAX_SEG_KEYS = 48_000_000
MAX_SEG_WIDE = 24_000_000


def _keys(name, n, type_="int32", kind="uniform", ascending=True):
    return {"name": name, "op": "keys", "n": n, "type": type_, "kind": kind,
            "ascending": ascending}


def _pairs(name, n, type_="int32", kind="uniform", ascending=True, values="index"):
    return {"name": name, "op": "pairs", "n": n, "type": type_, "kind": kind,
            "ascending": ascending, "values": values}


def _segments(name, nseg, lo, hi, type_="int32", ascending=True, op="segments", bounded=True):
    return {"name": name, "op": op, "nseg": nseg, "min_log2": lo, "max_log2": hi,
            "lengths_seed": 1506014460 + nseg, "type": type_, "kind": "uniform",
            "ascending": ascending, "bounded": bounded}


def listed():
    return [
        # a request of a thousand keys: one launch, all latency
        _keys("keys_1000", 1000),
        # the paper's workload, single arrays of 32-bit integers: a size
        # between one tile and the chip, the headline size, a size that is
        # not a power of two, and the largest size of the distribution sweep
        # (few distinct values, descending)
        _keys("keys_64k", 1 << 16),
        _keys("keys_10m", 10_000_000),
        _keys("keys_16m", 1 << 24),
        _keys("keys_64m_distinct16_desc", 1 << 26, kind="distinct16", ascending=False),
        # scores ranked from the best down, an odd length
        _keys("float32_1m_desc", 1_000_003, "float32", ascending=False),
        # 8-byte keys (identifiers, time stamps) and a stable argsort
        _keys("int64_16m", 1 << 24, "int64"),
        _pairs("argsort_16m", 1 << 24),
        # the batched workload: 8192 uneven arrays in one call, as keys and as
        # a per-segment argsort
        _segments("batch_8192", 8192, 0.0, 16.0),
        _segments("batch_8192_argsort", 8192, 0.0, 16.0, op="segment_pairs"),
        # one batch of the serving loop: a few requests of 2^8 .. 2^22 keys
        _segments("serving_batch_12", 12, 8.0, 22.0),
        # many short rows of 8-byte keys whose longest length the caller does
        # not know (no bound given)
        _segments("float64_rows_unbounded", 500, 0.0, 13.0, "float64", bounded=False),
    ]


def _log_size(rng, lo, hi):
    u = rng.uniform(lo, hi)
    if rng.random() < 0.25:
        return 1 << int(round(u))          # a power of two
    return int(round(2.0 ** u)) | (1 if rng.random() < 0.5 else 0)


def draw(rng):
    op = rng.choice(["keys", "keys", "keys", "keys64", "pairs", "segments", "segments",
                     "segment_pairs"])
    ascending = rng.random() < 0.5
    kind = rng.choice(["uniform", "uniform", "uniform", "sorted", "reverse", "distinct16", "equal"])
    if op == "keys":
        n = min(_log_size(rng, 8.0, 26.0), MAX_KEYS32)
        c = _keys("", n, rng.choice(["int32", "int32", "uint32", "float32"]), kind, ascending)
    elif op == "keys64":
        n = min(_log_size(rng, 8.0, 24.0), MAX_WIDE)
        c = _keys("", n, rng.choice(["int64", "uint64", "float64"]), kind, ascending)
    elif op == "pairs":
        n = min(_log_size(rng, 8.0, 24.0), MAX_WIDE)
        c = _pairs("", n, rng.choice(["int32", "uint32", "float32"]), kind, ascending,
                   rng.choice(["index", "uniform"]))
    else:
        wide = op == "segment_pairs" or rng.random() < 0.25
        type_ = rng.choice(["int32", "uint32", "float32"])
        if op == "segments" and wide:
            type_ = rng.choice(["int64", "uint64", "float64"])
        hi = rng.uniform(5.0, 22.0)
        lo = rng.uniform(0.0, hi / 2)
        most = MAX_SEG_WIDE if wide else MAX_SEG_KEYS
        mean = (2.0 ** hi - 2.0 ** lo) / ((hi - lo) * 0.6931471805599453)
        top = min(13.0, max(0.0, math.log2(most / (3.0 * mean))))
        nseg = max(1, min(8192, int(round(2.0 ** rng.uniform(0.0, top)))))
        c = _segments("", nseg, lo, hi, type_, ascending, op, rng.random() < 0.5)
        c["lengths_seed"] = rng.randrange(1 << 30)
        c["kind"] = kind if kind != "reverse" else "uniform"
        if int(_lengths(c).sum()) > most:
            return draw(rng)
    del c["name"]
    return c


def _lengths(case):
    """Segment lengths round(2**u), u uniform in [min_log2, max_log2]: part of
    the case, like n (the keys come from prepare's seed)."""
    u = W.unit_doubles(case["lengths_seed"], case["nseg"])
    u = case["min_log2"] + (case["max_log2"] - case["min_log2"]) * u
    return np.floor(np.exp2(u) + 0.5).astype(np.int64)


def _size(case):
    return int(_lengths(case).sum()) if case["op"].startswith("segment") else case["n"]


def _draw_uniform(type_, n, gen):
    """n keys: integers over their type's full range, floats normal."""
    if type_ in ("float32", "float64"):
        return torch.randn(n, generator=gen, device="cuda", dtype=getattr(torch, type_))
    if ELEM[type_] == 4:
        return torch.randint(-2**31, 2**31, (n,), generator=gen, device="cuda", dtype=torch.int32)
    return torch.randint(-2**63, 2**63 - 1, (n,), generator=gen, device="cuda",
                         dtype=torch.int64)


def _make_keys(case, n, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, type_ = case["kind"], case["type"]
    if kind == "distinct16":
        values = _draw_uniform(type_, 16, gen)
        return values[torch.randint(0, 16, (n,), generator=gen, device="cuda")]
    if kind == "equal":
        return _draw_uniform(type_, 1, gen).expand(n).contiguous()
    keys = _draw_uniform(type_, n, gen)
    if kind in ("sorted", "reverse"):
        return keys[_order(case, keys, None, None, ascending=kind == "sorted")]
    return keys


def prepare(case, seed):
    n = _size(case)
    src = _make_keys(case, n, seed)
    s = {"case": case, "src": src, "keys": torch.empty_like(src)}
    if case["op"].startswith("segment"):
        lens = _lengths(case)
        s["offsets"] = torch.from_numpy(W.offsets_from_lengths(lens)).cuda()
        s["bound"] = int(lens.max()) if case["bounded"] else 0
    if case["op"] in ("pairs", "segment_pairs"):
        if case["op"] == "segment_pairs":      # position inside its own segment
            starts = torch.repeat_interleave(s["offsets"][:-1], s["offsets"].diff())
            s["src_values"] = (torch.arange(n, device="cuda") - starts).to(torch.int32)
        elif case["values"] == "index":
            s["src_values"] = torch.arange(n, device="cuda", dtype=torch.int32)
        else:
            gen = torch.Generator(device="cuda")
            gen.manual_seed(seed + 1)
            s["src_values"] = torch.randint(-2**31, 2**31, (n,), generator=gen, device="cuda",
                                            dtype=torch.int32)
        s["values"] = torch.empty_like(s["src_values"])
    return s


def run(s):
    case, keys = s["case"], s["keys"]
    op, type_, asc = case["op"], case["type"], case["ascending"]
    keys.copy_(s["src"])
    if op == "keys":
        if ELEM[type_] == 8:
            B.bitonic_sort_keys64(keys, asc, type_)
        elif type_ == "int32":
            B.bitonic_sort_i32(keys, asc)
        else:
            B.bitonic_sort_keys(keys, asc, type_)
        return {"keys": keys}
    if op == "segments":
        B.bitonic_sort_segmented_keys(keys, s["offsets"], asc, type_, s["bound"])
        return {"keys": keys}
    s["values"].copy_(s["src_values"])
    if op == "pairs":
        B.bitonic_sort_pairs(keys, s["values"], asc, type_)
    else:
        B.bitonic_sort_segmented_pairs(keys, s["values"], s["offsets"], asc, type_, s["bound"])
    return {"keys": keys, "values": s["values"]}


def work(case):
    """Every key (and value) read once and written once."""
    n = _size(case)
    per = ELEM[case["type"]] + (4 if "pairs" in case["op"] else 0)
    off = 8 * (case["nseg"] + 1) if case["op"].startswith("segment") else 0
    return {"bytes": 2 * per * n + off, "flops": 0}


def _order(case, keys, values, segments, ascending):
    """Indices that put the keys in order: by segment, then by key, then by
    value, each with torch's stable sort."""
    k = keys
    if case["type"] == "uint32":
        k = keys.to(torch.int64) & 0xFFFFFFFF
    elif case["type"] == "uint64":
        k = keys ^ (-2**63)
    if values is None:
        at = torch.sort(k, stable=True, descending=not ascending).indices
    else:
        at = torch.sort(values, stable=True).indices
        at = at[torch.sort(k[at], stable=True, descending=not ascending).indices]
    if segments is not None:
        at = at[torch.sort(segments[at], stable=True).indices]
    return at


def exact(case, seed):
    s = prepare(case, seed)
    segments = None
    if "offsets" in s:
        lens = s["offsets"].diff()
        segments = torch.repeat_interleave(
            torch.arange(len(lens), device="cuda", dtype=torch.int32), lens)
    at = _order(case, s["src"], s.get("src_values"), segments, case["ascending"])
    keys = s["src"][at]
    out = {"keys": keys.double() if keys.is_floating_point() else keys}
    if "src_values" in s:
        out["values"] = s["src_values"][at]
    return out
