"""Checks that pick a code path by length, at lengths of the paths that the
shorter logs and batches of the other files do not reach: hash tables (up to
262,144 records), the sorting pipeline above, and the persistent digest kernel
(more work items than workgroups)."""
import numpy as np
import pytest

import oracle
import test_gpu_analyze as analyze
from gpu_helpers import compare
from paper_2601_12713_amd import workloads as W
from test_gpu_digest_forms import EDGES, host_views
from test_gpu_unused import EXPECT_UT, HAND_TRACES, check, padded, savings_trace, trace

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TABLES, SORTS = 5_000, 263_000


@pytest.mark.parametrize("total", [TABLES, SORTS])
@pytest.mark.parametrize("name", sorted(HAND_TRACES))
def test_hand_traces(odp, name, total):
    fg, _ = check(odp, padded(trace(HAND_TRACES[name]), total))
    assert [1 if f & odp.F_UT else 0 for f in fg[:len(HAND_TRACES[name])]] == EXPECT_UT[name]


@pytest.mark.parametrize("total", [TABLES, SORTS])
def test_savings_estimate(odp, total):
    _, rg = check(odp, padded(savings_trace(), total))
    assert rg["elim_ns"] == 29 and rg["span_ns"] == 90 + (total - 9) - 1
    ev = W.empty_events(total)
    ev["op"], ev["dst_dev"], ev["src_dev"] = W.H2D, 0, -1
    ev["src_addr"] = W.HOST_BASE + 64 * np.arange(total, dtype=np.uint64)
    ev["digest"] = np.arange(total, dtype=np.uint64)
    _, rg = check(odp, ev)
    assert rg["span_ns"] == 0 and rg["predicted_speedup"] == 1.0 and rg["ut_events"] == total
    ev["t_end"] = 5
    _, rg = check(odp, ev)
    assert rg["elim_ns"] == 5 * total and rg["predicted_speedup"] == float("inf")


WINDOW = 1024  # copies that the table form's forward search looks ahead


@pytest.mark.parametrize("gap", [1000, 1023, 1024, 1025, 1500])
@pytest.mark.parametrize("every", [1020, 1030, 4000])
def test_copies_left_open_by_the_search(odp, gap, every):
    """Chronological table logs whose next copy of a place lies `gap` copies on and
    whose kernels are `every` copies apart, on both sides of the window: copies
    with both beyond it are decided by the copies' table. Starts tie with the
    next kernel's on purpose."""
    n = 30_000
    ev = W.empty_events(n)
    k = np.arange(n)
    is_k = k % (every + 1) == every
    copy = np.cumsum(~is_k) - 1  # number of the copy
    ev["op"] = np.where(is_k, W.KERNEL, W.H2D)
    ev["src_dev"], ev["dst_dev"] = -1, 0
    ev["src_addr"] = W.HOST_BASE + 4096 * (copy % gap)
    ev["digest"] = k
    ev["t_start"] = np.cumsum(np.random.default_rng(gap).integers(0, 2, size=n)) + 1
    ev["t_end"] = ev["t_start"] + 1
    ev["bytes"] = 64
    # copies after each one that lie before the next kernel
    to_kernel = (every - 1) - k[~is_k] % (every + 1)
    last = k[~is_k] >= n - n % (every + 1)  # no kernel follows: unused at once
    undecided = int(np.sum((to_kernel >= WINDOW) & ~last)) if gap > WINDOW else 0
    assert (undecided > 0) == (gap > WINDOW and every > WINDOW)
    _, rg = check(odp, ev)
    assert 0 < rg["ut_events"]


@pytest.mark.parametrize("n", [4_500, 20_000, 300_000])
def test_calls_with_fixed_buffers(odp, n):
    """The same buffers again and again (launched, captured, replayed), with other
    records in them each time and other work between."""
    d_ev = torch.zeros(64 * n, dtype=torch.uint8, device="cuda")
    d_fl = torch.zeros(n, dtype=torch.uint8, device="cuda")
    d_rep = torch.zeros(odp.REPORT_BYTES, dtype=torch.uint8, device="cuda")
    for seed in range(5):
        ev, _, _ = W.tiny_trace(seed, n_events=n, n_devices=3, n_payloads=4, invalid_rate=0.001 if seed == 3 else 0.0)
        ev["digest"] = np.random.default_rng(seed).integers(0, 1 + n // (seed + 1), size=n)
        d_ev.copy_(torch.from_numpy(ev.view(np.uint8).reshape(-1).copy()))
        d_fl.fill_(0xAA)
        odp.analyze_trace(d_ev, d_fl, d_rep, n=n)
        torch.cuda.synchronize()
        compare(d_fl.cpu().numpy(), odp.report_to_dict(d_rep.cpu().numpy()), *oracle.analyze(ev))


@pytest.mark.parametrize("tx_share", [0.5, 0.02, 0.0, 1.0])
def test_digest_sort_keeps_only_transfers(odp, tx_share):
    analyze.test_digest_sort_keeps_only_transfers(odp, 270_000, tx_share)


@pytest.mark.parametrize("byte", [7, 3])
def test_long_runs_of_shared_low_bytes(odp, byte):
    analyze.test_long_runs_of_shared_low_bytes(odp, 300_000, byte)


def test_digests_sharing_low_bytes(odp):
    analyze.test_digests_sharing_low_bytes(odp, 300_000, 3)


@pytest.mark.parametrize("shifts", [[0], [1], [4], [0, 1, 4, 8, 15, 0, 64]])
def test_persistent_kernel(odp, shifts):
    """More node items than workgroups: every path edge at every kind of alignment,
    neighbours of different alignment in one queue; launch widths, launched and
    replayed; items claimed one and three at a time."""
    rng = np.random.default_rng(len(shifts) + shifts[0])
    sizes = [EDGES[i % len(EDGES)] for i in range(len(EDGES) * len(shifts))]
    host, dev, ptrs = host_views(rng, sizes, [shifts[(i + i // len(EDGES)) % len(shifts)] for i in range(len(sizes))])
    want = [oracle.d64(h) for h in host]
    times = 2 + 8192 // sum(-(-s // 262144) for s in sizes if s > 4096)  # 8,192 node items at least
    order = rng.permutation(len(sizes) * times) % len(sizes)
    n = order.size
    dp = torch.tensor(np.array(ptrs, dtype=np.uint64)[order].view(np.int64), device="cuda")
    ds = torch.tensor(np.array(sizes, dtype=np.int64)[order], device="cuda")
    want = np.array(want, dtype=np.uint64)[order]
    out = torch.empty(n, dtype=torch.int64, device="cuda")
    saved = odp.get_tuning()
    try:
        for use_graph, bpc, chunk in ((1, 4, 1), (0, 1, 1), (1, 8, 3)):
            odp.set_tuning(blocks_per_cu=bpc, use_graph=use_graph, chunk_nodes=chunk)
            for _ in range(3):  # launched, captured, replayed
                out.fill_(-1)
                odp.digest_buffers(dp, ds, out)
                assert (out.cpu().numpy().view(np.uint64) == want).all(), (use_graph, bpc, chunk)
    finally:
        odp.set_tuning(**saved)
    out.fill_(-1)
    odp.digest_buffers_noalloc(dp[:16384], ds[:16384], out)
    assert (out[:min(n, 16384)].cpu().numpy().view(np.uint64) == want[:16384]).all()
    assert odp.device_status() == 0
