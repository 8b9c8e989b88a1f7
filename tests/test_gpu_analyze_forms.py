"""The analysis at the log lengths where its form changes, against the oracle:
every flag and every report field, bit-exact."""
import numpy as np
import pytest

import oracle
from paper_2601_12713_amd import workloads as W

from gpu_helpers import analyze_gpu, compare

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def random_log(seed, n, devices=3, digests=40, places=12, invalid=0.0, kernels=0.12, allocs=0.25, tie=0.3, long_kernels=False):
    """A random log with few keys (every rule fires), ties, and records out of order when invalid > 0."""
    rng = np.random.default_rng(seed)
    ev = W.empty_events(n)
    u = rng.random(n)
    op = np.where(u < kernels, W.KERNEL, np.where(u < kernels + allocs, rng.choice([W.ALLOC, W.DELETE], size=n),
                                                  rng.choice([W.H2D, W.D2H, W.D2D], size=n)))
    ev["op"] = op
    ev["digest"] = rng.integers(0, digests, size=n).astype(np.uint64) * np.uint64(0x9E3779B97F4A7C15)
    ev["src_dev"], ev["dst_dev"] = rng.integers(-1, devices, size=n), rng.integers(-1, devices, size=n)
    ev["src_addr"] = W.HOST_BASE + rng.integers(0, places, size=n) * 4096
    ev["dst_addr"] = W.DEV_BASE + rng.integers(0, places, size=n) * 4096
    ev["bytes"] = rng.choice([64, 128], size=n)
    ev["t_start"] = np.cumsum(rng.integers(0, 10, size=n) * (rng.random(n) >= tie)) + 50
    ev["t_end"] = ev["t_start"] + rng.integers(0, 400 if long_kernels else 8, size=n)
    bad = rng.random(n) < invalid
    back = bad & (rng.random(n) < 0.5)  # before its predecessor: what follows may start earlier than what was
    ev["t_start"][back] -= rng.integers(1, 50, size=int(back.sum())).astype(np.uint64)
    ev["op"][bad & ~back] = 9
    return ev


def check(odp, ev):
    fr, rr = oracle.analyze(ev)
    fg, rg = analyze_gpu(odp, ev)
    compare(fg, rg, fr, rr)
    return fg, rg


@pytest.mark.parametrize("n", [512, 513, 640, 1023, 1024, 1025, 2047, 3001])
@pytest.mark.parametrize("invalid", [0.0, 0.02])
def test_walked_logs(odp, n, invalid):
    check(odp, random_log(n, n, invalid=invalid))
    check(odp, random_log(n + 1, n, devices=10, digests=n, places=n, invalid=invalid, long_kernels=True))
    check(odp, random_log(n + 2, n, devices=1, digests=2, places=1, invalid=invalid, kernels=0.002))


@pytest.mark.parametrize("kind", ["no kernels", "kernels only", "allocations only", "all rejected", "one digest"])
def test_walked_one_class(odp, kind):
    n = 3000
    ev = random_log(7, n, kernels=1.0 if kind == "kernels only" else 0.0 if kind == "no kernels" else 0.1,
                    allocs=1.0 if kind == "allocations only" else 0.2, digests=1 if kind == "one digest" else 40)
    if kind == "allocations only":
        ev["op"] = np.where(np.arange(n) % 3 == 0, W.ALLOC, W.DELETE)
    if kind == "all rejected":
        ev["op"] = 0
    check(odp, ev)


@pytest.mark.parametrize("n", [4095, 4096, 4097])
def test_last_walked_length(odp, n):
    check(odp, random_log(n, n, digests=n // 4, places=300, invalid=0.001))


def test_walked_calls_alternate(odp):
    """Calls on one stream share the workspace: logs of other lengths between, under capture and replayed."""
    logs = [random_log(100 + k, m) for k, m in enumerate((600, 4000, 3000, 30000))]
    want = [oracle.analyze(ev) for ev in logs]
    for k in (0, 1, 3, 2, 0, 3, 1):
        fg, rg = analyze_gpu(odp, logs[k])
        compare(fg, rg, *want[k])
    s = torch.cuda.Stream()
    odp.reserve(max_events=4000, stream=s)
    ev = logs[1]
    d_ev = torch.from_numpy(ev.view(np.uint8).reshape(-1).copy()).to("cuda")
    d_fl = torch.zeros(len(ev), dtype=torch.uint8, device="cuda")
    d_rep = torch.zeros(odp.REPORT_BYTES, dtype=torch.uint8, device="cuda")
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        odp.analyze_trace(d_ev, d_fl, d_rep, stream=s, n=len(ev))
    for _ in range(3):
        d_fl.fill_(0xAA)
        g.replay()
        torch.cuda.synchronize()
        compare(d_fl.cpu().numpy(), odp.report_to_dict(d_rep.cpu().numpy()), *want[1])
        odp.analyze_trace(d_ev, d_fl, d_rep, n=len(ev))


@pytest.mark.parametrize("n", [4097, 6143, 6144, 6145, 16385, 50000])
@pytest.mark.parametrize("invalid", [0.0, 0.01])
def test_table_logs(odp, n, invalid):
    """Groups in hash tables: few hot keys, as many keys as records, long
    stretches without kernels, all endpoints."""
    check(odp, random_log(n, n, invalid=invalid))
    check(odp, random_log(n + 1, n, devices=10, digests=n, places=n, invalid=invalid, long_kernels=True))
    check(odp, random_log(n + 2, n, devices=1, digests=3, places=1, invalid=invalid, kernels=0.0005))
    check(odp, random_log(n + 3, n, devices=2, digests=500, places=3000, invalid=invalid, kernels=0.6, allocs=0.3))
    check(odp, random_log(n + 4, n, devices=1, digests=n // 3, places=400, invalid=invalid, kernels=0.001, allocs=0.9))


def test_table_log_one_digest(odp):
    """One group over every workgroup: the carries are looked up past 64 wavefronts."""
    n = 40000
    ev = random_log(3, n, digests=1, kernels=0.01, allocs=0.01)
    check(odp, ev)
    ev["op"] = W.H2D  # one direction, one receiver
    ev["src_dev"], ev["dst_dev"] = -1, 0
    check(odp, ev)
    ev["op"][:-1] = W.D2H  # the return leg is the last record
    ev["src_dev"][:-1], ev["dst_dev"][:-1] = 0, -1
    check(odp, ev)


@pytest.mark.parametrize("n", [262143, 262144, 262145])
def test_last_table_length(odp, n):
    check(odp, random_log(n, n, devices=4, digests=n // 8, places=2000, invalid=0.0))
    check(odp, random_log(n, n, devices=4, digests=n // 8, places=2000, invalid=0.0005))


def test_keys_that_collide_in_the_tables(odp):
    """Digests and addresses that are multiples of large powers of two."""
    n = 9000
    ev = random_log(11, n, digests=n, places=n, kernels=0.02)
    k = np.arange(n, dtype=np.uint64)
    ev["digest"] = (k % 3000) << np.uint64(40)
    ev["src_addr"] = (k % 700) << np.uint64(33)
    ev["dst_addr"] = (k % 900) << np.uint64(50)
    check(odp, ev)


@pytest.mark.parametrize("kind", ["random", "out of order", "shared low bytes", "one digest", "few kernels", "all ones"])
def test_sorted_logs(odp, kind):
    """The sorting pipeline, just above the last table length."""
    n = 262145 + 4096 + 7
    ev = random_log(n, n, devices=3, digests=n // 8, places=2000, invalid=0.001 if kind == "out of order" else 0.0,
                    kernels=0.0002 if kind == "few kernels" else 0.1, long_kernels=kind == "out of order")
    k = np.arange(n, dtype=np.uint64)
    if kind == "shared low bytes":  # long runs of equal low bytes holding several digests
        ev["digest"] = (k % 5) << np.uint64(48) | (k % 7) << np.uint64(40) | (k % 3000) // np.uint64(1000)
    if kind == "one digest":
        ev["digest"] = 77
    if kind == "all ones":
        ev["digest"] = np.where(k % 3 == 0, np.uint64(2**64 - 1), k // np.uint64(4) << np.uint64(8) | np.uint64(255))
    check(odp, ev)


@pytest.mark.parametrize("kind", ["all single", "pairs among single", "self transfers", "crowded byte", "long ranges", "one byte varies"])
def test_single_digests_are_dropped(odp, kind):
    """Digests that occur once leave the sort after its first pass, by ranges of their lowest byte."""
    n = 300_001
    ev = random_log(n, n, devices=10 if kind == "pairs among single" else 3, digests=40, places=2000,
                    kernels=0.05, allocs=0.05 if kind in ("crowded byte", "long ranges") else 0.25)
    k = np.arange(n, dtype=np.uint64)
    digest = k * np.uint64(0x9E3779B97F4A7C15)  # each once
    if kind in ("pairs among single", "crowded byte", "long ranges"):
        digest = np.where(k % 5 == 0, digest[n // 2], digest)
        digest[n // 2:] = np.where(k[n // 2:] % 3 == 0, digest[:n - n // 2], digest[n // 2:])
    if kind == "crowded byte":  # more than 2^17 transfers in one range
        digest = digest & ~np.uint64(255) | np.where(k % 10 == 0, k % np.uint64(256), np.uint64(9))
    if kind == "long ranges":   # 6 ranges around and above the elements held per thread
        digest = digest & ~np.uint64(255) | np.where(k % 7 == 0, np.uint64(3), k % np.uint64(6))
    if kind == "self transfers":
        ev["src_dev"] = ev["dst_dev"] = 1
        digest = np.where(k % 50 == 0, np.uint64(5), digest)
    if kind == "one byte varies":
        digest = k % np.uint64(256)
    ev["digest"] = digest
    check(odp, ev)


@pytest.mark.parametrize("kind", ["one device", "ten devices", "few kernels", "long kernels", "ties", "one place", "kernel every other", "rejected"])
def test_unused_transfers_by_span(odp, kind):
    """Copies decided inside their 512 records, and what crosses to the next ones."""
    n = 262_145 + 513
    ev = random_log(n, n, devices=10 if kind == "ten devices" else 1, digests=n, places=1 if kind == "one place" else 50,
                    kernels={"few kernels": 0.0005, "kernel every other": 0.5}.get(kind, 0.02), allocs=0.05,
                    tie=0.97 if kind == "ties" else 0.3)
    if kind == "long kernels":
        k = np.flatnonzero(ev["op"] == W.KERNEL)[::40]
        ev["t_end"][k] += np.uint64(3000)
    if kind == "rejected":
        ev["t_end"][n // 2] = ev["t_start"][n // 2] - np.uint64(1)
    check(odp, ev)


@pytest.mark.parametrize("n", [4097, 4097 + 63, 20000])
@pytest.mark.parametrize("hot", [1, 2, 9, 300])
def test_table_logs_of_hot_digests(odp, n, hot):
    """A wavefront's lanes want the same few empty slots at once, beside fresh digests."""
    ev = random_log(n + hot, n, digests=n, kernels=0.02, allocs=0.05)
    k = np.arange(n, dtype=np.uint64)
    ev["digest"] = np.where(k % 7 == 3, ev["digest"], (k % np.uint64(hot)) * np.uint64(0xC2B2AE3D27D4EB4F))
    check(odp, ev)


def lifetimes(n, arrays, devices, gap, seed):
    """ALLOC/DELETE records of `arrays` addresses per device, each freed `gap` of
    its own kind later, between other records; some frees come twice."""
    rng = np.random.default_rng(seed)
    ev = W.empty_events(n)
    i = np.arange(n)
    rec = rng.random(n)
    ev["op"] = np.where(rec < 0.03, W.KERNEL, np.where(rec < 0.06, W.H2D, np.where((i // gap) % 2 == 0, W.ALLOC, W.DELETE)))
    slot = i % gap % arrays if seed % 2 else (gap - 1 - i % gap) % arrays
    slot = np.where(rng.random(n) < 0.02, rng.integers(0, arrays, size=n), slot)
    ev["src_dev"], ev["dst_dev"] = -1, slot % devices
    ev["src_addr"] = W.HOST_BASE + 4096 * (slot % 37)
    ev["dst_addr"] = W.DEV_BASE + 4096 * slot
    ev["bytes"] = 64 + 64 * (slot % 3)
    ev["digest"] = rng.integers(0, 1 << 40, size=n)
    ev["t_start"] = np.cumsum(rng.integers(0, 5, size=n))
    ev["t_end"] = ev["t_start"] + rng.integers(0, 5, size=n)
    return ev


@pytest.mark.parametrize("n", [4097, 70_000, 262_144])
@pytest.mark.parametrize("arrays,gap", [(1, 1), (10, 10), (300, 300), (255, 1024), (2000, 2000), (1 << 17, 60_000)])
def test_table_logs_lifetimes(odp, n, arrays, gap):
    """Neighbours of a group inside 64 positions, inside a chunk, in the chunk
    before and far chunks; chunks of 256 to 1,024 positions."""
    for seed in (1, 2):
        check(odp, lifetimes(n, arrays, 3, gap, seed))


@pytest.mark.parametrize("n", [5000, 66_000, 262_144])
@pytest.mark.parametrize("places", [1, 40, 3000, 50_000])
@pytest.mark.parametrize("rejected", [False, True])
def test_table_logs_far_copies(odp, n, places, rejected):
    """Copies whose next copy or kernel lies beyond the forward search, in logs
    with and without a rejected record: the copies' table, read backwards."""
    rng = np.random.default_rng(n + places)
    ev = W.empty_events(n)
    ev["op"] = np.where(np.arange(n) % 3001 == 3000, W.KERNEL, np.where(rng.random(n) < 0.02, W.D2H, W.H2D))
    ev["src_dev"] = np.where(ev["op"] == W.D2H, 0, -1)
    ev["dst_dev"] = np.where(ev["op"] == W.D2H, -1, rng.integers(0, 2, size=n))
    ev["src_addr"] = W.HOST_BASE + 4096 * rng.integers(0, places, size=n)
    ev["digest"] = rng.integers(0, n, size=n)
    ev["t_start"] = np.cumsum(rng.integers(0, 2, size=n)) + 10
    ev["t_end"] = ev["t_start"] + rng.integers(0, 3, size=n)
    ev["bytes"] = 64
    if rejected:
        ev["op"][n // 3] = 9
    fg, rg = check(odp, ev)
    assert 0 < rg["ut_events"]


@pytest.mark.parametrize("n", [4097, 20_000, 262_144])
@pytest.mark.parametrize("hosts", [1, 3, 300])
def test_table_logs_repeated_allocations(odp, n, hosts):
    """Few (host address, device, bytes) keys: a wavefront's pairs share one
    entry of the repeated-allocation table; frees in either order."""
    for seed in (1, 2):
        ev = lifetimes(n, 500, 2, 700, seed)
        slot = ((ev["dst_addr"] - np.uint64(W.DEV_BASE)) // np.uint64(4096)).astype(np.int64)
        ev["src_addr"] = W.HOST_BASE + 4096 * (slot % hosts)
        ev["bytes"] = 64
        check(odp, ev)


@pytest.mark.parametrize("kernels", [1, 2, 2047, 2048, 2049, 4097, 9000])
def test_table_logs_out_of_order_kernels(odp, kernels):
    """Logs that are not chronological: the kernels of a device in sorted tiles
    of 2,048, the last one partly filled; one end at the type's largest value."""
    n = 6000 + 2 * kernels
    ev = random_log(kernels, n, devices=2, digests=n, places=200, invalid=0.0, kernels=0.0)
    at = np.sort(np.random.default_rng(kernels).choice(n, size=kernels + 5, replace=False))
    ev["op"][at] = W.KERNEL
    ev["dst_dev"][at] = 0
    ev["dst_dev"][at[::kernels // 5 + 1]] = 1
    ev["t_end"][at] += np.random.default_rng(kernels).integers(0, 300, size=at.size).astype(np.uint64)
    half = n // 2  # the clock jumps back once
    ev["t_start"][half:] -= ev["t_start"][half] - ev["t_start"][half // 2]
    ev["t_end"][half:] -= np.minimum(ev["t_end"][half:], ev["t_end"][half] - ev["t_start"][half // 2])
    ev["t_end"] = np.maximum(ev["t_end"], ev["t_start"])
    ev["t_end"][at[-1]] = np.uint64(2**64 - 1)
    fg, rg = check(odp, ev)
    assert rg["status"] == 1


@pytest.mark.parametrize("places", [1, 90, 5000])
@pytest.mark.parametrize("every", [509, 515, 1023, 4001])
def test_sorted_logs_far_kernels(odp, every, places):
    """The sorting pipeline's forward search: a copy's kernel just inside and past
    its window of listed copies, its next copy before and behind what is searched."""
    n = 262_145 + 3 * every
    rng = np.random.default_rng(every * places)
    ev = W.empty_events(n)
    ev["op"] = np.where(np.arange(n) % every == every - 1, W.KERNEL, W.H2D)
    ev["src_dev"], ev["dst_dev"] = -1, 0
    ev["src_addr"] = W.HOST_BASE + 4096 * rng.integers(0, places, size=n)
    ev["digest"] = rng.integers(0, n, size=n)
    ev["t_start"] = np.cumsum(rng.integers(0, 2, size=n)) + 10
    ev["t_end"] = ev["t_start"] + rng.integers(0, 2, size=n)
    ev["bytes"] = 64
    check(odp, ev)


@pytest.mark.parametrize("share", [7, 8, 9, 33, 64])
@pytest.mark.parametrize("devices", [1, 10])
def test_sorted_logs_many_kernels(odp, share, devices):
    """Rounds of 64 records with few and many kernels among the copies, some of
    them still running at later copies."""
    n = 262_145 + 700
    ev = random_log(share, n, devices=devices, digests=n, places=30, kernels=share / 64, allocs=0.1, long_kernels=share == 9)
    check(odp, ev)


@pytest.mark.parametrize("places", [1, 2, 3, 4, 7])
@pytest.mark.parametrize("kernels", [0.0, 0.05, 0.4])
def test_sorted_logs_near_copies(odp, places, kernels):
    """Copies of a few places in turn or at random: the next copy one, two or more
    lanes on, in the next round, and across the span; places of equal hash bits."""
    n = 262_145 + 700
    rng = np.random.default_rng(places)
    for order in ("turn", "random"):
        ev = W.empty_events(n)
        ev["op"] = np.where(rng.random(n) < kernels, W.KERNEL, np.where(rng.random(n) < 0.1, W.D2H, W.H2D))
        d2h = ev["op"] == W.D2H
        ev["src_dev"], ev["dst_dev"] = np.where(d2h, 0, -1), np.where(d2h, -1, rng.integers(0, 2, size=n))
        place = np.arange(n) % places if order == "turn" else rng.integers(0, places, size=n)
        ev["src_addr"] = W.HOST_BASE + (place.astype(np.uint64) << np.uint64(12))
        ev["digest"] = np.arange(n)
        ev["t_start"] = np.cumsum(rng.integers(0, 3, size=n)) + 10
        ev["t_end"] = ev["t_start"] + rng.integers(0, 6, size=n)
        ev["bytes"] = 64
        check(odp, ev)
