"""Digest launch forms against the oracle, bit-exact, at the sizes where each
form's choice of path changes."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LEAF, NODE = 4096, 262144
EDGES = [0, 1, 31, 32, 100, LEAF - 1, LEAF, LEAF + 1, 2 * LEAF, 3 * LEAF + 17, 16 * LEAF, 17 * LEAF + 5, 48 * LEAF + 1,
         NODE - 1, NODE, NODE + 1, 2 * NODE + 7, 65 * NODE + 4099]


def host_views(rng, sizes, shifts):
    """(host bytes, device arena, device addresses) of buffers at 256-byte slots plus their shifts."""
    slot = [(s + 16 + 511) // 256 * 256 for s in sizes]
    base = np.concatenate([[0], np.cumsum(slot)])
    host = rng.integers(0, 256, size=int(base[-1]), dtype=np.uint8)
    dev = torch.from_numpy(host).to("cuda")
    off = [int(b) + sh for b, sh in zip(base, shifts)]
    return [host[o:o + s] for o, s in zip(off, sizes)], dev, [dev.data_ptr() + o for o in off]


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 300])
def test_host_descriptors_share_launches(odp, n):
    """One call over n host descriptors: a launch holds 128 of them."""
    rng = np.random.default_rng(n)
    small = [s for s in EDGES if s <= NODE]
    sizes = [EDGES[i] if i < len(EDGES) else small[int(rng.integers(0, len(small)))] for i in range(n)]
    host, dev, ptrs = host_views(rng, sizes, [int(x) for x in rng.choice([0, 0, 0, 1, 4, 8], size=n)])
    want = [oracle.d64(h) for h in host]
    out = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    for _ in range(2):  # the second call finds the first one's tickets and tree slots
        out.fill_(-1)
        odp.digest_buffers_plain(ptrs, sizes, out)
        assert out.cpu().numpy().view(np.uint64).tolist() == want


def test_host_descriptors_captured(odp):
    """Captured launches keep their descriptors: replays after the host arrays are gone."""
    rng = np.random.default_rng(5)
    sizes = EDGES * 9
    host, dev, ptrs = host_views(rng, sizes, [0] * len(sizes))
    want = [oracle.d64(h) for h in host]
    out = torch.full((len(sizes),), -1, dtype=torch.int64, device="cuda")
    s = torch.cuda.Stream()
    odp.digest_buffers_plain(ptrs, sizes, out, s)  # sizes the workspace of the stream
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        odp.digest_buffers_plain(ptrs, sizes, out, s)
    del ptrs
    for _ in range(3):
        out.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert out.cpu().numpy().view(np.uint64).tolist() == want


@pytest.mark.parametrize("shift", [1, 2, 3, 4, 6, 8, 12, 15])
def test_array_sections(odp, shift):
    """Buffers that start inside an allocation: 4-byte aligned ones are staged
    like whole allocations, the rest word by word; every path edge in each form."""
    rng = np.random.default_rng(shift)
    host, dev, ptrs = host_views(rng, EDGES, [shift] * len(EDGES))
    want = [oracle.d64(h) for h in host]
    n = len(EDGES)
    out = torch.full((n,), -1, dtype=torch.int64, device="cuda")
    dp = torch.tensor(np.array(ptrs, dtype=np.uint64).view(np.int64), device="cuda")
    ds = torch.tensor(np.array(EDGES, dtype=np.int64), device="cuda")
    for form in (lambda: odp.digest_buffers(dp, ds, out), lambda: odp.digest_buffers_noalloc(dp, ds, out),
                 lambda: odp.digest_buffers_plain(ptrs, EDGES, out),
                 lambda: [odp.digest_buffers_plain(ptrs[i:i + 1], EDGES[i:i + 1], out[i:]) for i in range(n)]):
        out.fill_(-1)
        form()
        assert out.cpu().numpy().view(np.uint64).tolist() == want


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 8191, 8192, 8193])
@pytest.mark.parametrize("split", [0, 65536])
def test_plan_sizes(odp, n, split):
    """Both sides of the one-launch plan's limits, with and without medium
    nodes; calls with new arguments launch directly, repeats replay a graph."""
    keep = odp.get_tuning()
    odp.set_tuning(split_bytes=split)
    try:
        calls = []
        for seed in (n, n + 1):
            rng = np.random.default_rng(seed)
            sizes = rng.integers(0, 6000, size=n)
            some = rng.choice(n, size=min(n, 40), replace=False)
            sizes[some] = [EDGES[i % len(EDGES)] for i in range(some.size)]
            host, dev, ptrs = host_views(rng, [int(s) for s in sizes], [0] * n)
            dp = torch.tensor(np.array(ptrs, dtype=np.uint64).view(np.int64), device="cuda")
            ds = torch.tensor(sizes.astype(np.int64), device="cuda")
            calls.append((dp, ds, torch.empty(n, dtype=torch.int64, device="cuda"), oracle.d64_many(host), dev))
        for k in (0, 1, 0, 0, 0, 1, 1):
            dp, ds, out, want, _ = calls[k]
            out.fill_(-1)
            odp.digest_buffers(dp, ds, out)
            assert (out.cpu().numpy().view(np.uint64) == want).all()
        assert odp.device_status() == odp.ODP_OK
    finally:
        odp.set_tuning(**keep)
