"""The work that a user of this library has it do, as measurable cases.

Every case goes through the package's public entry points.  A sort is in place, so
a pass first copies the unsorted records over the work buffer with the library's
own streaming copy and then sorts them: a pass is "sort these records", and can be
repeated.  Keys are unsigned bit patterns in int32 / int64 tensors and the payload is
the record's index, as in the package's workloads.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2607_05302_amd as radsort

DEV = "cuda:0"
ALIGN = 256  # bytes; the planes of a record buffer start on this boundary
KEY_T = {4: torch.int32, 8: torch.int64}


def _sort(name, n, kb, vb, dist, block, keep_ws, shared=False, op="sort"):
    c = {"op": op, "n": n, "key_bytes": kb, "payload_bytes": vb, "dist": dist, "block": block,
         "keep_ws": keep_ws, "shared": shared}
    return {"name": name, **c} if name else c


def _segments(name, count, lo, hi, kb, vb):
    c = {"op": "segments", "count": count, "lo_log2": lo, "hi_log2": hi, "key_bytes": kb,
         "payload_bytes": vb}
    return {"name": name, **c} if name else c


def _resort(name, n, block):
    c = {"op": "resort", "n": n, "block": block}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one short list, called as the README shows it (the library finds its own
        # workspace): what a call costs when the data is next to nothing
        _sort("tiny_pairs", 1500, 4, 4, "uniform", 1024, False),
        # a list that fits any cache, odd length, workspace kept by the program
        _sort("pairs_49k", 49275, 4, 4, "uniform", 1024, True),
        # the plain array of 2^20 uint32 keys with an index, b = 1024
        _sort("pairs_1m", 1 << 20, 4, 4, "uniform", 1024, True),
        # a request of the serving loop: uint64 keys with a uint32 index, the GPU shared
        # with other requests, workspace in the server's arena
        _sort("serve_u64_3m", 3000017, 8, 4, "uniform", 1024, True, shared=True),
        # the README's example size, default options
        _sort("pairs_16m", (1 << 24) + 3, 4, 4, "uniform", 1024, False),
        # the large array of the benchmark: 2^28 pairs, b = 2048
        _sort("pairs_256m", 1 << 28, 4, 4, "uniform", 2048, True),
        # the structured uint64 inputs: Zipf keys without payload, b = 4096
        _sort("zipf_u64_256m", 1 << 28, 8, 0, "zipf", 4096, True),
        # the same family with an index payload: only the low 20 bits differ
        _sort("low20_u64_64m", (1 << 26) - 5, 8, 4, "low20", 2048, True),
        # a batch of short arrays (each fits one workgroup's LDS)
        _segments("batch_short", 4096, 6, 13, 4, 4),
        # a batch of uneven arrays, the sizes of the batched benchmark
        _segments("batch_mixed", 512, 10, 22, 4, 4),
        # new keys written in place through the block table, sorted again without
        # finalize or setup, and read out in logical order
        _resort("resort_64m", 1 << 26, 2048),
        # the out-of-place sort, for programs that have the memory
        _sort("oop_10m", 10000019, 4, 4, "uniform", 1024, True, op="oop"),
    ]


def _log_size(rng, lo, hi):
    """A size log-uniform in [2^lo, 2^hi], odd as often as not."""
    return max(2, int(2.0 ** rng.uniform(lo, hi)))


def draw(rng):
    """One more case of the same ranges: sizes over their logarithm, both key widths,
    every payload width, the distributions and block sizes the workloads use."""
    kind = rng.choice(["sort", "sort", "sort", "sort", "sort", "oop", "segments", "resort"])
    if kind == "segments":
        hi = rng.uniform(11, 21)
        kb, vb = rng.choice([(4, 4), (4, 4), (4, 0), (8, 4), (8, 0)])
        # at most about 2^26 elements in all
        count = min(4096, max(8, int(2.0 ** (26 - hi) * (hi - 6) * math.log(2.0))))
        return _segments("", rng.randrange(max(4, count // 4), count + 1), 6.0, hi, kb, vb)
    if kind == "resort":
        return _resort("", _log_size(rng, 16, 26), rng.choice([1024, 2048]))
    kb = rng.choice([4, 4, 8])
    vb = rng.choice([0, 4, 4, 8])
    n = _log_size(rng, 6, 28 if kb + vb <= 8 else 27)
    block = 1024 if n < 1 << 22 else rng.choice([1024, 2048, 4096])
    dist = rng.choice(["uniform", "uniform", "uniform", "zipf", "low20", "sorted", "equal"])
    shared = kind == "sort" and rng.random() < 0.3
    return _sort("", n, kb, vb, dist, block, shared or rng.random() < 0.7, shared, kind)


# ---- inputs ------------------------------------------------------------------------------


def _uniform(g, n, kb):
    lim = 31 if kb == 4 else 63
    return torch.randint(-(1 << lim), (1 << lim) - 1, (n,), generator=g, dtype=KEY_T[kb],
                         device=DEV)


def _keys(dist, n, kb, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    if dist == "uniform":
        return _uniform(g, n, kb)
    if dist == "equal":  # one key everywhere
        return _uniform(g, 1, kb).expand(n).contiguous()
    if dist == "low20":  # only the low 20 bits random
        return _uniform(g, n, kb) & ((1 << 20) - 1)
    if dist == "sorted":  # already ascending (unsigned)
        top = -(1 << (8 * kb - 1))
        return torch.sort(_uniform(g, n, kb) ^ top).values ^ top
    if dist == "zipf":  # Zipf(s = 1.1) over 2^16 distinct values
        distinct = 1 << 16
        values = _uniform(g, distinct, kb)
        cdf = torch.cumsum(torch.arange(1, distinct + 1, dtype=torch.float64, device=DEV) ** -1.1, 0)
        cdf /= cdf[-1].clone()
        out = torch.empty(n, dtype=values.dtype, device=DEV)
        for lo in range(0, n, 1 << 25):
            hi = min(n, lo + (1 << 25))
            u = torch.rand(hi - lo, generator=g, dtype=torch.float64, device=DEV)
            out[lo:hi] = values[torch.searchsorted(cdf, u, right=True).clamp_(max=distinct - 1)]
        return out
    raise ValueError(dist)


def _planes(n, kb, vb):
    """A record buffer and its key and payload planes."""
    at = (n * kb + ALIGN - 1) // ALIGN * ALIGN
    buf = torch.empty(at + n * vb, dtype=torch.uint8, device=DEV)
    keys = buf[:n * kb].view(KEY_T[kb])
    vals = buf[at:at + n * vb].view(KEY_T[vb]) if vb else None
    return buf, keys, vals


def _sizes(case, seed):
    """Array sizes of a batch, log-uniform; the same for every seed, so that a case is
    always the same amount of work."""
    r = np.random.RandomState(0x5E6 + case["count"])
    u = r.uniform(case["lo_log2"], case["hi_log2"], case["count"])
    return np.floor(2.0 ** u).astype(np.int64)


def _multiplier(step):
    """An odd multiplier per step (uint32), as a signed int."""
    m = (0x9E3779B1 * (2 * step + 1)) & 0xFFFFFFFF | 1
    return m - (1 << 32) if m >= 1 << 31 else m


def prepare(case, seed):
    op = case["op"]
    if op == "resort":
        n, b = case["n"], case["block"]
        keys = _keys("uniform", n, 4, seed)
        # the payload identifies the record, and a program's records differ by seed
        vals = torch.arange(n, dtype=torch.int32, device=DEV) + (seed & 0xFFFF)
        ws = torch.empty(radsort.workspace_bytes(n, 4, 4, 8, b), dtype=torch.uint8, device=DEV)
        st = radsort.State(keys, vals, digit_bits=8, block_elems=b, workspace=ws)
        tk, tv, bb = st.planes()
        size = 2 * st.sigma * bb * 4
        t_keys = ws[tk - ws.data_ptr():tk - ws.data_ptr() + size].view(torch.int32)
        t_vals = ws[tv - ws.data_ptr():tv - ws.data_ptr() + size].view(torch.int32)
        t_vals.zero_()
        st.setup()
        for _ in range(st.nt):
            st.round()
        return {"op": op, "st": st, "keys": keys, "vals": vals, "t_keys": t_keys,
                "t_vals": t_vals, "ws": ws, "step": 0}
    kb, vb = case["key_bytes"], case["payload_bytes"]
    s = {"op": op}
    if op == "segments":
        sizes = _sizes(case, seed)
        offsets = np.concatenate([[0], np.cumsum(sizes)]).astype(np.uint64)
        n = int(offsets[-1])
        s["offsets"] = offsets
        s["offsets_dev"] = torch.from_numpy(offsets.view(np.int64)).to(DEV)
        s["ws"] = torch.empty(radsort.segments_workspace_bytes(offsets, kb, vb),
                              dtype=torch.uint8, device=DEV)
        dist = "uniform"
    else:
        n, dist = case["n"], case["dist"]
        s["block"], s["shared"] = case["block"], case["shared"]
        s["ws"] = None
        if case["keep_ws"]:
            nbytes = (radsort.oop_workspace_bytes(n, kb, vb, 8, case["block"]) if op == "oop" else
                      radsort.workspace_bytes(n, kb, vb, 8, case["block"], shared=case["shared"]))
            s["ws"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    s["src"], k, v = _planes(n, kb, vb)
    k.copy_(_keys(dist, n, kb, seed))
    if vb:
        v.copy_(torch.arange(n, dtype=KEY_T[vb], device=DEV))
    s["buf"], s["keys"], s["vals"] = _planes(n, kb, vb)
    return s


def run(s):
    if s["op"] == "resort":
        m, st = _multiplier(s["step"]), s["st"]
        s["step"] += 1
        torch.mul(s["vals"], m, out=s["keys"])
        torch.mul(s["t_vals"], m, out=s["t_keys"])
        st.restart()
        for _ in range(st.nt):
            st.round()
        return list(st.logical())
    radsort.copy_(s["buf"], s["src"])
    if s["op"] == "sort":
        radsort.sort_(s["keys"], s["vals"], block_elems=s["block"], workspace=s["ws"],
                      shared=s["shared"])
    elif s["op"] == "oop":
        radsort.oop_sort_(s["keys"], s["vals"], block_elems=s["block"], workspace=s["ws"])
    else:
        radsort.sort_segments_(s["keys"], s["vals"], s["offsets"], workspace=s["ws"],
                               offsets_dev=s["offsets_dev"])
    return [s["keys"], s["vals"]]


def work(case):
    """Each record read once and written once; comparisons are no floating point."""
    if case["op"] == "resort":
        return {"bytes": 2.0 * case["n"] * 8, "flops": 0.0}
    n = int(_sizes(case, 0).sum()) if case["op"] == "segments" else case["n"]
    return {"bytes": 2.0 * n * (case["key_bytes"] + case["payload_bytes"]), "flops": 0.0}


def _stable(keys, kb):
    """Order of a stable ascending sort of unsigned keys."""
    wide = keys.to(torch.int64) & 0xFFFFFFFF if kb == 4 else keys ^ -(1 << 63)
    return torch.sort(wide, stable=True)[1]


def exact(case, seed):
    """The sorted records from torch's stable sort of 64-bit keys (on the GPU)."""
    if case["op"] == "resort":
        n = case["n"]
        vals = torch.arange(n, dtype=torch.int32, device=DEV) + (seed & 0xFFFF)
        keys = vals * _multiplier(0)
        at = _stable(keys, 4)
        return [keys[at], vals[at]]
    kb, vb = case["key_bytes"], case["payload_bytes"]
    if case["op"] == "segments":
        sizes = _sizes(case, seed)
        n = int(sizes.sum())
        keys = _keys("uniform", n, kb, seed)
        seg = torch.repeat_interleave(torch.arange(len(sizes), device=DEV),
                                      torch.from_numpy(sizes).to(DEV))
        at = _stable(keys, kb)
        at = at[torch.sort(seg[at], stable=True)[1]]
    else:
        n = case["n"]
        keys = _keys(case["dist"], n, kb, seed)
        at = _stable(keys, kb)
    return [keys[at], at.to(KEY_T[vb]) if vb else None]
