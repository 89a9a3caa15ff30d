"""The sorts a program asks of this library, as measurable cases.

A case is a dict of plain values.  ``op`` names the entry point:

  keys      mms.sort            uint32 / int32 keys
  pairs     mms.sort_pairs      stable (32-bit key, input index) pairs
  keys64    mms.sort64          uint64 / int64 keys
  pairs64   mms.sort_pairs64    stable (64-bit key, 64-bit index) pairs
  batch     mms.segmented_sort  many arrays in one call, keys or stable pairs
  served    mms.Server          a burst of requests of mixed kinds and sizes

``signed`` is the key order (int32 / int64 or uint32 / uint64).  ``keep``
says what the caller holds between calls: with it the output and the
workspace are allocated once, as a program that sorts in a loop does; without
it every call allocates them, as a single call does.  ``family`` is the key
distribution: uniform over all values, sixteen distinct values, a sorted
sequence with random swaps (n / 100 of them), or a sorted sequence
interleaved with stride 64.
"""
import math
import random

import numpy as np
import torch

import paper_1702_07961_amd as mms

FAMILIES = ("uniform", "sixteen", "nearly", "stride64")


def listed():
    return [
        # one small array: a single workgroup sorts it, the call itself is what counts
        {"name": "keys_1000", "op": "keys", "n": 1000, "family": "uniform", "signed": True, "keep": False},
        # a few tiles, an odd size: launches and dependent steps on a mostly idle chip
        {"name": "keys_40961", "op": "keys", "n": 40_961, "family": "uniform", "signed": False, "keep": False},
        # the plain sort of 2^20 keys
        {"name": "keys_2p20", "op": "keys", "n": 1 << 20, "family": "uniform", "signed": False, "keep": True},
        # between the latency-bound and the throughput-bound sizes
        {"name": "keys_6300007", "op": "keys", "n": 6_300_007, "family": "uniform", "signed": True, "keep": True},
        # the headline: 10^8 uniform keys
        {"name": "keys_1e8", "op": "keys", "n": 100_000_000, "family": "uniform", "signed": False, "keep": True},
        # re-sorting data that is almost in order
        {"name": "keys_1e8_nearly", "op": "keys", "n": 100_000_000, "family": "nearly", "signed": True, "keep": True},
        # group-by style keys with few values, an odd mid size, one call
        {"name": "pairs_300007_sixteen", "op": "pairs", "n": 300_007, "family": "sixteen", "signed": False,
         "keep": False},
        # the large stable key-value sort (an argsort of 2^27 keys)
        {"name": "pairs_2p27", "op": "pairs", "n": 1 << 27, "family": "uniform", "signed": False, "keep": True},
        # 8-byte keys
        {"name": "keys64_1e8", "op": "keys64", "n": 100_000_000, "family": "uniform", "signed": False, "keep": True},
        # 8-byte keys with 8-byte values, an odd size
        {"name": "pairs64_33554467", "op": "pairs64", "n": 33_554_467, "family": "uniform", "signed": True,
         "keep": True},
        # thousands of arrays in one call, sizes log-uniform in [2^8, 2^20]
        {"name": "batch_4096", "op": "batch", "segments": 4096, "lo": 8, "hi": 20, "pairs": False, "sizes": 1,
         "family": "uniform", "signed": False, "keep": True},
        # a burst of requests through the serving loop, half of them pairs
        {"name": "served_40", "op": "served", "requests": 40, "lo": 10, "hi": 22, "sizes": 2, "family": "uniform",
         "signed": False},
    ]


def _log_uniform(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    op = rng.choice(("keys", "keys", "keys", "pairs", "pairs", "keys64", "pairs64", "batch", "batch", "served"))
    family = rng.choice(("uniform", "uniform") + FAMILIES)
    signed = rng.random() < 0.5
    if op == "batch":
        lo, hi = rng.choice(((6, 12), (8, 16), (8, 20)))
        segs = _log_uniform(rng, 16, 512 if hi == 20 else 4096)
        return {"op": op, "segments": segs, "lo": lo, "hi": hi, "pairs": rng.random() < 0.5,
                "sizes": rng.randrange(1 << 20), "family": "uniform", "signed": signed, "keep": True}
    if op == "served":
        return {"op": op, "requests": rng.randrange(16, 41), "lo": 10, "hi": rng.choice((16, 20, 22)),
                "sizes": rng.randrange(1 << 20), "family": "uniform", "signed": signed}
    top = {"keys": 100_000_000, "pairs": 1 << 27, "keys64": 100_000_000, "pairs64": 33_554_467}[op]
    return {"op": op, "n": _log_uniform(rng, 256, top), "family": family, "signed": signed,
            "keep": rng.random() < 0.5}


# ---- inputs ------------------------------------------------------------------------
def _sizes(case, count):
    rng = random.Random(case["sizes"])
    return [_log_uniform(rng, 1 << case["lo"], 1 << case["hi"]) for _ in range(count)]


def _keys(case, n, gen, bits):
    """n keys of the case's family, as an int32 / int64 device tensor holding
    the keys' bits."""
    dt = torch.int32 if bits == 32 else torch.int64
    family = case["family"]
    if family == "uniform":
        if bits == 32:
            return torch.randint(-(1 << 31), 1 << 31, (n,), generator=gen, device="cuda", dtype=torch.int64).to(dt)
        hi = torch.randint(-(1 << 31), 1 << 31, (n,), generator=gen, device="cuda", dtype=torch.int64)
        hi <<= 32
        hi += torch.randint(0, 1 << 32, (n,), generator=gen, device="cuda", dtype=torch.int64)
        return hi
    if family == "sixteen":
        v = torch.randint(0, 16, (n,), generator=gen, device="cuda", dtype=torch.int64)
        return (v * (0x11111111 if bits == 32 else 0x1111111111111111)).to(dt)
    if family == "nearly":
        # the start differs with the seed, so that the values do too
        start = int(torch.randint(0, 1 << 20, (1,), generator=gen, device="cuda").item())
        x = torch.arange(start, start + n, device="cuda", dtype=dt)
        k = n // 100
        if k:
            at = torch.randperm(n, generator=gen, device="cuda")[:2 * k]
            i, j = at[:k], at[k:]
            a = x[i].clone()
            x[i] = x[j]
            x[j] = a
        return x
    start = int(torch.randint(0, 1 << 20, (1,), generator=gen, device="cuda").item())
    i = torch.arange(n, device="cuda", dtype=torch.int64)
    return (start + (i % 64) * ((n + 63) // 64) + i // 64).to(dt)


def _gen(seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    return gen



def _offsets(case):
    return np.concatenate(([0], np.cumsum(_sizes(case, case["segments"])))).astype(np.uint64)


def _requests(case, seed):
    """[(keys, values or None)] of a served case: every second request is pairs."""
    gen = _gen(seed)
    reqs = []
    for q, n in enumerate(_sizes(case, case["requests"])):
        k = _keys(case, n, gen, 32)
        reqs.append((k, torch.arange(n, device="cuda", dtype=torch.int32) if q % 2 else None))
    return reqs


def prepare(case, seed):
    op = case["op"]
    st = {"case": case, "op": op, "signed": case["signed"]}
    if op == "served":
        st["reqs"] = _requests(case, seed)
        st["server"] = mms.Server(budget_bytes=2 << 30)
        st["open"] = []
        return st
    if op == "batch":
        st["off"] = _offsets(case)
        n = int(st["off"][-1])
    else:
        n = case["n"]
    wide = op in ("keys64", "pairs64")
    pairs = op in ("pairs", "pairs64") or bool(case.get("pairs"))
    keys = _keys(case, n, _gen(seed), 64 if wide else 32)
    st["keys"] = keys
    st["values"] = torch.arange(n, device="cuda", dtype=keys.dtype) if pairs else None
    st["out_k"] = st["out_v"] = st["ws"] = None
    if case["keep"]:
        st["out_k"] = torch.empty_like(keys)
        st["out_v"] = torch.empty_like(keys) if pairs else None
        if op == "batch":
            need = mms.segmented_workspace_bytes(st["off"], pairs)
        else:
            need = mms.workspace_bytes(n, pairs, wide)
        st["ws"] = torch.empty(max(need, 1), device="cuda", dtype=torch.uint8)
    return st


# ---- one pass ----------------------------------------------------------------------
def run(st):
    op, signed = st["op"], st["signed"]
    if op == "keys":
        return mms.sort(st["keys"], out=st["out_k"], i32=signed, workspace=st["ws"])
    if op == "pairs":
        return mms.sort_pairs(st["keys"], st["values"], out_keys=st["out_k"], out_values=st["out_v"], i32=signed,
                              workspace=st["ws"])
    if op == "keys64":
        return mms.sort64(st["keys"], out=st["out_k"], i64=signed, workspace=st["ws"])
    if op == "pairs64":
        return mms.sort_pairs64(st["keys"], st["values"], out_keys=st["out_k"], out_values=st["out_v"], i64=signed,
                                workspace=st["ws"])
    if op == "batch":
        return mms.segmented_sort(st["keys"], st["off"], values=st["values"], out_keys=st["out_k"],
                                  out_values=st["out_v"], i32=signed, workspace=st["ws"])
    srv = st["server"]
    stream = torch.cuda.current_stream()
    for t in st["open"]:              # the results of the pass before have been read
        srv.release(t, stream)
    st["open"] = [srv.submit(k, v, i32=signed) for k, v in st["reqs"]]
    out = []
    for t in st["open"]:
        r = srv.wait(t)
        out.append(r.keys)
        if r.values is not None:
            out.append(r.values)
    return out


# ---- what a pass cannot do without ----------------------------------------------------
def work(case):
    op = case["op"]
    if op == "served":
        n = sum(s * (2 if q % 2 else 1) for q, s in enumerate(_sizes(case, case["requests"])))
        return {"bytes": 8 * n, "flops": 0}
    if op == "batch":
        return {"bytes": 8 * sum(_sizes(case, case["segments"])) * (2 if case["pairs"] else 1), "flops": 0}
    size = {"keys": 4, "pairs": 8, "keys64": 8, "pairs64": 16}[op]
    return {"bytes": 2 * size * case["n"], "flops": 0}


# ---- the same results from torch in 64 bits --------------------------------------------
def _sorted(keys, signed, with_order):
    """Stably sorted keys (same dtype) and, if asked, their input positions."""
    k = keys.to(torch.int64)
    if not signed:
        k = (k & 0xFFFFFFFF) if keys.dtype == torch.int32 else k ^ (-(1 << 63))
    order = torch.sort(k, stable=True)[1]
    return keys[order], order if with_order else None


def exact(case, seed):
    op, signed = case["op"], case["signed"]
    if op == "served":
        out = []
        for k, v in _requests(case, seed):
            ks, order = _sorted(k, signed, v is not None)
            out.append(ks)
            if v is not None:
                out.append(v[order])
        return out
    if op == "batch":
        off = [int(x) for x in _offsets(case)]
        keys = _keys(case, off[-1], _gen(seed), 32)
        vals = torch.empty_like(keys) if case["pairs"] else None
        for a, b in zip(off[:-1], off[1:]):
            ks, order = _sorted(keys[a:b], signed, case["pairs"])
            keys[a:b] = ks
            if case["pairs"]:
                vals[a:b] = (order + a).to(torch.int32)
        return (keys, vals) if case["pairs"] else keys
    pairs = op in ("pairs", "pairs64")
    keys = _keys(case, case["n"], _gen(seed), 64 if op.endswith("64") else 32)
    ks, order = _sorted(keys, signed, pairs)
    return (ks, order.to(keys.dtype)) if pairs else ks
