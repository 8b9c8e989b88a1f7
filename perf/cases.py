"""The work that a user of this framework has it do, as measurable cases.

Each case is one call (one session for the server) of a public entry point of
``paper_2601_12713_amd.odp``: the content digest in its three forms, the trace
analysis, its comparison mode, and the request server. Sizes are those of the
repository's own workloads (``workloads.py``, ``bench.py``, the autotuner's
batch) or lie inside their ranges. Every output is a whole number (digests,
flags, counts, sums) except the server's predicted speedup, so there is no
64-bit reference to be further from.
"""
import math

import numpy as np
import torch

from paper_2601_12713_amd import odp
from paper_2601_12713_amd import workloads as W

DEV = "cuda:0"


def listed():
    return [
        # One transfer hashed as it is logged: one buffer, one call (the smallest call there is).
        {"name": "plain_one", "kind": "plain", "n": 1, "lo": 100000, "hi": 100000, "shift": 0},
        # The buffers of a small program, one call with host descriptors (the plain-small workload's sizes).
        {"name": "plain_mix", "kind": "plain", "n": 64, "lo": 4096, "hi": 262144, "shift": 0},
        # One large fp64 array of 2^25 elements (the large-arrays workload).
        {"name": "plain_large", "kind": "plain", "n": 1, "lo": 1 << 28, "hi": 1 << 28, "shift": 0},
        # A handful of small variables digested together, device descriptors.
        {"name": "batch_small", "kind": "batch", "n": 64, "lo": 64, "hi": 65536, "total": 0, "shift": 0},
        # The autotuner's batch: 20,000 buffers, log-uniform sizes scaled to 8e9 bytes.
        {"name": "batch_mixed", "kind": "batch", "n": 20000, "lo": 64, "hi": 1 << 24, "total": 8000000000, "shift": 0},
        # Array sections: transfers of a[lo:len] start at an element of an array, not at an allocation,
        # so their addresses are multiples of the element (8 bytes here) only.
        {"name": "batch_sections", "kind": "batch", "n": 2000, "lo": 4096, "hi": 1 << 23, "total": 0, "shift": 8},
        # Many scalars, structs and short arrays in the form that allocates nothing.
        {"name": "noalloc_many", "kind": "noalloc", "n": 4096, "lo": 1, "hi": 16384, "total": 0, "shift": 0},
        # Logs: a small program's (the plain-small workload's length), a longer run's, and the trace at scale.
        {"name": "trace_1k", "kind": "analyze", "n": 1000, "slots": 64, "devices": 1, "rejected": 0},
        {"name": "trace_100k", "kind": "analyze", "n": 100000, "slots": 2000, "devices": 1, "rejected": 0},
        {"name": "trace_10m", "kind": "analyze", "n": 10675000, "slots": 100000, "devices": 1, "rejected": 0},
        # Three devices and the host: the analysis with the pairs of the literal Algorithm 2 beside it.
        {"name": "alg2_200k", "kind": "alg2", "n": 200000, "slots": 4000, "devices": 3, "rejected": 0},
        # A short-lived server that is handed a backlog of requests and drained.
        {"name": "serve_backlog", "kind": "serve", "n": 2000, "lo": 4096, "hi": 1 << 20},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["plain", "batch", "batch", "noalloc", "analyze", "analyze", "analyze", "alg2", "serve"])
    if kind == "plain":
        n = _log_int(rng, 1, 128)
        hi = _log_int(rng, 64, (1 << 28) // n)
        lo = max(1, hi // rng.choice([1, 4, 64]))
        return {"kind": kind, "n": n, "lo": lo, "hi": hi, "shift": rng.choice([0, 0, 4, 8])}
    if kind in ("batch", "noalloc"):
        n = _log_int(rng, 8, 16384)
        hi = _log_int(rng, 256, min(1 << 24, 16000000000 // n))
        lo = max(1, hi // rng.choice([4, 64, 4096]))
        return {"kind": kind, "n": n, "lo": lo, "hi": hi, "total": 0, "shift": rng.choice([0, 0, 1, 4, 8])}
    if kind == "analyze":
        n = _log_int(rng, 32, 8000000)
        return {"kind": kind, "n": n, "slots": _log_int(rng, 4, max(8, n // 16)), "devices": rng.choice([1, 1, 2, 4, 8]),
                "rejected": rng.choice([0, 0, 0, 0, 3])}
    if kind == "alg2":
        n = _log_int(rng, 500, 1000000)
        return {"kind": kind, "n": n, "slots": _log_int(rng, 16, max(32, n // 16)), "devices": rng.choice([2, 3, 7]),
                "rejected": 0}
    return {"kind": kind, "n": _log_int(rng, 100, 4000), "lo": 4096, "hi": _log_int(rng, 1 << 15, 1 << 22)}


# ---------------------------------------------------------------------------
# Inputs.
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _sizes(case):
    """Buffer sizes of a digest case: the same for every seed (they set the work)."""
    rng = np.random.default_rng(1000003 * case["n"] + case["lo"] + 7 * case["hi"])
    n, lo, hi = case["n"], case["lo"], case["hi"]
    if case.get("total"):
        return W.batch_sizes(case["n"] + 81, n, lo, hi, case["total"])[0].astype(np.int64)
    if lo == hi:
        return np.full(n, lo, dtype=np.int64)
    if case["kind"] == "plain":
        return rng.integers(lo, hi + 1, size=n)
    return np.floor(np.exp(rng.uniform(math.log(lo), math.log(hi + 1), size=n))).astype(np.int64)


def _buffers(case, seed):
    """One arena of random bytes and the buffers' offsets in it: 256-byte aligned
    (allocations), or at a random multiple of `shift` bytes (sections of arrays
    of such elements)."""
    sizes = _sizes(case)
    slot = (sizes + 2 * 256 - 1) // 256 * 256
    off = np.concatenate([[0], np.cumsum(slot)[:-1]]).astype(np.int64)
    if case["shift"]:
        rng = np.random.default_rng(seed)
        off = off + case["shift"] * rng.integers(0, 256 // case["shift"], size=sizes.size)
    words = int(slot.sum()) // 8
    arena = torch.empty(words, dtype=torch.int64, device=DEV)
    g, step = _gen(seed), 1 << 27
    for a in range(0, words, step):
        m = min(step, words - a)
        arena[a:a + m].random_(generator=g)
    return arena, off + arena.data_ptr(), sizes


def _zipf(g, n_items, size):
    w = torch.arange(1, n_items + 1, dtype=torch.float64, device=DEV) ** -1.1
    cdf = torch.cumsum(w, 0)
    u = torch.rand(size, generator=g, dtype=torch.float64, device=DEV) * cdf[-1]
    return torch.searchsorted(cdf, u).clamp_(max=n_items - 1)


def _trace(case, seed):
    """A log of n records with the shape of the trace-at-scale workload, made on
    the GPU: variables by a finite Zipf(1.1); 15% of the map records re-send the
    variable's last host-to-device content, 3% form H2D-D2H-H2D triples of one
    content, 2% ALLOC/DELETE pairs (half around a KERNEL), the rest move fresh
    contents; a KERNEL after every 16 map records. With several devices each
    variable has a home device and some copies go device to device. `rejected`
    records get an end before their start."""
    n, devices, g = case["n"], case["devices"], _gen(seed)
    units = n  # more than enough; the log is cut at n records
    u = torch.rand(units, generator=g, device=DEV)
    edges = torch.tensor([0.4065, 0.8135, 0.9685, 0.97885, 0.9896], device=DEV)  # 3% and 2% of records, by units
    kind = torch.searchsorted(edges, u)  # 0 fresh H2D, 1 fresh D2H / D2D, 2 re-send, 3 triple, 4 used pair, 5 unused pair
    slot = _zipf(g, case["slots"], units)
    dig = torch.empty(units, dtype=torch.int64, device=DEV).random_(generator=g)
    dig = dig ^ (torch.randint(0, 2, (units,), generator=g, device=DEV) << 63)
    # re-sends take the content of the latest earlier H2D of their variable
    order = torch.sort(slot, stable=True).indices
    ks, ss = kind[order], slot[order]
    at = torch.arange(units, device=DEV)
    last = torch.cummax(torch.where((ks == 0) | (ks == 3), at, -1), 0).values
    prev = torch.cat([last.new_full((1,), -1), last[:-1]])
    src = torch.where((prev >= 0) & (ss[prev.clamp(min=0)] == ss), order[prev.clamp(min=0)], -1)
    source = torch.empty_like(src)
    source[order] = src
    kind = torch.where((kind == 2) & (source < 0), torch.zeros_like(kind), kind)
    dig = torch.where(kind == 2, dig[source.clamp(min=0)], dig)
    del order, ks, ss, at, last, prev, src, source
    # expand the units into records
    maps = torch.tensor([1, 1, 1, 3, 2, 2], device=DEV)[kind]
    end = torch.cumsum(maps, 0)
    own = maps + (kind == 4)
    length = own + end // 16 - (end - maps) // 16
    start = torch.cumsum(length, 0) - length
    of = torch.repeat_interleave(torch.arange(units, device=DEV), length)[:n]
    pos = torch.arange(n, device=DEV) - start[of]
    k, s, periodic = kind[of], slot[of], pos >= own[of]
    table = torch.tensor([[W.H2D, 0, 0], [W.D2H, 0, 0], [W.H2D, 0, 0], [W.H2D, W.D2H, W.H2D],
                          [W.ALLOC, W.KERNEL, W.DELETE], [W.ALLOC, W.DELETE, 0]], device=DEV)
    op = torch.where(periodic, W.KERNEL, table[k, pos.clamp(max=2)])
    home = s % devices
    sd, dd = torch.full_like(s, -1), home.clone()
    if devices > 1:
        d2d = (k == 1) & ~periodic & (torch.rand(n, generator=g, device=DEV) < 0.3)
        op = torch.where(d2d, W.D2D, op)
        sd, dd = torch.where(d2d, home, sd), torch.where(d2d, (home + 1) % devices, dd)
    d2h = op == W.D2H
    sd, dd = torch.where(d2h, home, sd), torch.where(d2h, -1, dd)
    is_k = op == W.KERNEL
    nbytes = torch.exp(torch.rand(case["slots"], generator=g, dtype=torch.float64, device=DEV)
                       * math.log((1 << 24) / 8) + math.log(8)).long()[s]
    nbytes = torch.where(is_k, 0, nbytes)
    host, devm = W.HOST_BASE + s * (1 << 20), W.DEV_BASE + s * (1 << 20)
    gap = 1 + (-1000.0 * torch.log1p(-torch.rand(n, generator=g, dtype=torch.float64, device=DEV))).long()
    dur = 5000 + nbytes // 25
    t_end = torch.cumsum(gap + dur, 0)
    ev = torch.empty((n, 8), dtype=torch.int64, device=DEV)
    ev[:, 0] = torch.where((op >= W.H2D) & (op <= W.D2D), dig[of], 0)
    ev[:, 1] = torch.where(is_k, 0, torch.where(sd >= 0, devm, host))
    ev[:, 2] = torch.where(is_k, 0, torch.where(dd >= 0, devm, host))
    ev[:, 3], ev[:, 4], ev[:, 5], ev[:, 6] = nbytes, t_end - dur, t_end, 0x403000 + (k << 4)
    ev[:, 7] = (sd & 0xFFFF) | ((dd & 0xFFFF) << 16) | (op << 32)
    if case["rejected"]:
        bad = torch.randint(0, n, (case["rejected"],), generator=g, device=DEV)
        ev[bad, 5] = ev[bad, 4] - 1
    return ev


def prepare(case, seed):
    kind = case["kind"]
    odp.load()
    if kind in ("plain", "batch", "noalloc"):
        arena, ptrs, sizes = _buffers(case, seed)
        out = torch.zeros(sizes.size, dtype=torch.int64, device=DEV)
        if kind == "plain":
            return {"kind": kind, "arena": arena, "ptrs": ptrs.astype(np.uint64), "sizes": sizes.astype(np.uint64), "out": out}
        return {"kind": kind, "arena": arena, "ptrs": torch.from_numpy(ptrs).to(DEV),
                "sizes": torch.from_numpy(sizes).to(DEV), "out": out}
    if kind in ("analyze", "alg2"):
        n = case["n"]
        st = {"kind": kind, "n": n, "ev": _trace(case, seed), "flags": torch.zeros(n, dtype=torch.uint8, device=DEV),
              "report": torch.zeros(odp.REPORT_BYTES, dtype=torch.uint8, device=DEV)}
        if kind == "alg2":
            st["rx"] = torch.zeros(n, dtype=torch.int32, device=DEV)
            st["pairs"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        return st
    arena = torch.empty((1 << 28) // 8, dtype=torch.int64, device=DEV).random_(generator=_gen(seed)).view(torch.uint8)
    s = W.ServingSchedule(seed=seed, n=case["n"], rate=100000.0, lo=case["lo"], hi=case["hi"], arena=arena)
    return {"kind": kind, "n": case["n"], "arena": arena, "events": s.events, "ptrs": s.payload_ptrs(),
            "bytes": s.payload_bytes, "arrival": np.zeros(case["n"], dtype=np.uint64)}


def run(st):
    kind = st["kind"]
    if kind == "plain":
        return odp.digest_buffers_plain(st["ptrs"], st["sizes"], st["out"])
    if kind == "batch":
        return odp.digest_buffers(st["ptrs"], st["sizes"], st["out"])
    if kind == "noalloc":
        return odp.digest_buffers_noalloc(st["ptrs"], st["sizes"], st["out"])
    if kind == "analyze":
        odp.analyze_trace(st["ev"], st["flags"], st["report"], n=st["n"])
        return {"flags": st["flags"], "report": st["report"]}
    if kind == "alg2":
        odp.analyze_trace_alg2(st["ev"], st["flags"], st["report"], st["rx"], st["pairs"], n=st["n"])
        return {"flags": st["flags"], "report": st["report"], "rx": st["rx"], "pairs": st["pairs"]}
    # every request has arrived; which tick takes which request (and so what is
    # known early) depends on timing, the drained flags, report and log do not
    srv = odp.Server(max_events=st["n"], budget_bytes=1 << 30)
    try:
        srv.run(st["events"], st["ptrs"], st["bytes"], st["arrival"])
        _, flags, report = srv.drain()
        return {"flags": flags, "report": report, "log": srv.log()}
    finally:
        srv.close()


def work(case):
    kind = case["kind"]
    if kind in ("plain", "batch", "noalloc"):
        return {"bytes": int(_sizes(case).sum()) + 8 * case["n"], "flops": 0}
    if kind == "analyze":
        return {"bytes": 65 * case["n"] + odp.REPORT_BYTES, "flops": 0}
    if kind == "alg2":
        return {"bytes": 69 * case["n"] + odp.REPORT_BYTES + 8, "flops": 0}
    # 64-byte records in and out, and the payloads (0.91 of the records move a log-uniform slice)
    mean = (case["hi"] - case["lo"]) / math.log(case["hi"] / case["lo"])
    return {"bytes": int(case["n"] * (129 + 0.91 * mean)), "flops": 0}
