"""Served ticks on both sides of the length from which a tick's records are
grouped instead of walked: flags known before the drain, and drained, against
the oracle."""
import numpy as np
import pytest

import oracle

from gpu_helpers import compare
from test_gpu_analyze_forms import random_log
from test_gpu_serve import check_known

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("max_tick", [63, 64, 65, 192, 1023, 1024])
@pytest.mark.parametrize("kind", ["few keys", "many keys", "one key", "rejected"])
def test_tick_lengths(odp, max_tick, kind):
    n = 3 * max_tick + 17
    few = kind == "few keys"
    ev = random_log(max_tick, n, devices=10 if kind == "many keys" else 2, digests=1 if kind == "one key" else 20 if few else n,
                    places=1 if kind == "one key" else 6 if few else n // 2, invalid=0.03 if kind == "rejected" else 0.0)
    srv = odp.Server(max_events=n, budget_bytes=64 << 20, max_tick=max_tick)
    zero = np.zeros(n, dtype=np.uint64)
    _, stats = srv.run(ev, zero, zero, zero)
    known, fl, rep = srv.drain()
    srv.close()
    fo, ro = oracle.analyze(ev)
    compare(fl, rep, fo, ro)
    check_known(known, fo, ev)
    assert stats["max_tick"] <= max_tick


def test_drain_waits_for_the_default_stream(odp):
    """Output arrays that the default stream is still filling when the drain is
    called hold the drain's results afterwards, not the fill."""
    n = 400
    ev = random_log(5, n, devices=2, digests=50, places=20)
    srv = odp.Server(max_events=n, budget_bytes=64 << 20)
    zero = np.zeros(n, dtype=np.uint64)
    srv.run(ev, zero, zero, zero)
    known = torch.empty(n, dtype=torch.uint8, device="cuda")
    flags = torch.empty(n, dtype=torch.uint8, device="cuda")
    rep = torch.empty(odp.REPORT_BYTES, dtype=torch.uint8, device="cuda")
    a = torch.ones((4096, 4096), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    for _ in range(20):  # some milliseconds of work in front of the fills
        a = a @ a
    for out in (known, flags, rep):
        out.fill_(0xEE)
    assert odp.load().odp_server_drain(srv._h, *(t.data_ptr() for t in (known, flags, rep))) == odp.ODP_OK
    torch.cuda.synchronize()
    srv.close()
    fo, ro = oracle.analyze(ev)
    compare(flags.cpu().numpy(), odp.report_to_dict(rep.cpu().numpy()), fo, ro)
    check_known(known.cpu().numpy(), fo, ev)


@pytest.mark.parametrize("max_tick", [1, 2, 13, 31, 32, 33])
@pytest.mark.parametrize("kind", ["few keys", "kernels", "rejected", "waiting windows"])
def test_short_ticks(odp, max_tick, kind):
    """Ticks on both sides of the length up to which one wavefront takes all
    records; with more waiting windows than a workgroup has threads."""
    n = 4000 if kind == "waiting windows" else 40 * max_tick + 5
    ev = random_log(max_tick, n, devices=10 if kind == "kernels" else 2, digests=20, places=n if kind == "waiting windows" else 6,
                    invalid=0.03 if kind == "rejected" else 0.0, kernels=0.5 if kind == "kernels" else 0.05,
                    allocs=0.9 if kind == "waiting windows" else 0.25)
    if kind == "waiting windows":  # each address allocated, then freed; the frees end far behind the log's middle
        k = np.arange(n)
        pair = (ev["op"] != 6) & (k % 8 != 7)
        ev["op"] = np.where(pair, np.where(k % 2 == 0, 1, 5), ev["op"])
        ev["dst_dev"] = np.where(pair, 0, ev["dst_dev"])
        ev["dst_addr"] = np.where(pair, 4096 * (k // 2), ev["dst_addr"])
        late = int(ev["t_start"][-1]) - 3
        ev["t_end"] = np.where(pair & (k % 2 == 1) & (k < 3800), np.maximum(late - k % 50, ev["t_end"].astype(np.int64)), ev["t_end"])
    srv = odp.Server(max_events=n, budget_bytes=64 << 20, max_tick=max_tick)
    zero = np.zeros(n, dtype=np.uint64)
    _, stats = srv.run(ev, zero, zero, zero)
    known, fl, rep = srv.drain()
    srv.close()
    fo, ro = oracle.analyze(ev)
    compare(fl, rep, fo, ro)
    check_known(known, fo, ev)
    assert stats["max_tick"] == max_tick
    if kind == "waiting windows":
        assert rep["n_alloc_pairs"] > 1200 and rep["n_invalid"] == 0
