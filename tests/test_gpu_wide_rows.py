"""Rows that walk blocks pad themselves and rows that are filled first: widths
on both sides of the line (96 slots; more blocks than most SIMDs hold; outputs
past the last-level cache), plain, allocation-free, backward, batched and served.
Against the queue dispatch and the one-thread-per-walk batch, bit for bit, and
nothing outside the rows."""
import numpy as np
import pytest

from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu

# (walks, width): blocks 1, 2, 600 and 601, and 327,680 slots a lane's worth;
# long rows over 600 blocks and 601, and from 4,096 slots on over 192 and 193, or
# 400 and 401
SHAPES = [(1, 96), (1, 97), (65, 96), (65, 99), (65, 100), (65, 5000), (3000, 300), (38_400, 100),
          (38_401, 100), (40_000, 523), (40_000, 525), (209_000, 100), (210_000, 101),
          (38_401, 3071), (38_401, 3072), (12_288, 4096), (12_289, 4096),
          (25_600, 4097), (25_601, 4097)]


def _graph(torch, tw, directed):
    rng = np.random.default_rng(9)
    V, n = 500, 9000
    g = tw.Graph(V, directed=directed)
    g.ingest_batch(*to_dev(torch, rng.integers(0, V - 3, n).astype(np.int32),
                           rng.integers(0, V, n).astype(np.int32),
                           np.sort(rng.integers(0, 4000, n)).astype(np.int64)))
    return g


def _guarded(torch, W, L):
    n = torch.full((W * L + 8,), 7, dtype=torch.int32, device="cuda")
    t = torch.full((W * L + 8,), 7, dtype=torch.int64, device="cuda")
    return n, t, (n[4:4 + W * L].view(W, L), t[4:4 + W * L].view(W, L),
                  torch.full((W,), 7, dtype=torch.int32, device="cuda"))


@pytest.mark.parametrize("W,L", SHAPES)
@pytest.mark.parametrize("direction", ["forward", "backward"])
def test_plain_rows(W, L, direction):
    torch, tw = gpu_or_skip()
    g = _graph(torch, tw, direction == "forward")
    starts = torch.arange(W, dtype=torch.int32, device="cuda") % 500
    kw = dict(hop_bias="linear", start_mode="node", start_nodes=starts, seed=L)
    ref = g.sample_walks(W, L, dispatch="queue", direction=direction, **kw)
    for call in ("plain", "noalloc") if direction == "forward" else ("plain",):
        n, t, out = _guarded(torch, W, L)
        if call == "plain":
            g.sample_walks(W, L, out=out, dispatch="full_walk", direction=direction, **kw)
        else:
            g.sample_walks_noalloc(W, L, out, **kw)
        g.sync()
        for a, b in zip(out, ref):
            assert torch.equal(a, b), call
        for x in (n, t):
            assert bool((x[:4] == 7).all()) and bool((x[4 + W * L:] == 7).all())
    g.close()


@pytest.mark.parametrize("W,L", SHAPES)
def test_batch_rows(W, L):
    torch, tw = gpu_or_skip()
    g = _graph(torch, tw, False)
    biases = [("uniform", 0.0, 1.0, 1.0), ("linear", 0.0, 1.0, 1.0), ("exponential", 400.0, 1.0, 1.0)]
    lim = torch.full((W,), L, dtype=torch.int32, device="cuda")
    lim[::3] = max(1, L - 5)
    for rows in (None, g.row_offsets(lim)):
        kw = dict(max_lens=lim, seed=2, ragged=rows is not None, rows=rows)
        ref = g.sample_walks_batch(W, L, biases, dispatch="full_walk", **kw)
        out = g.sample_walks_batch(W, L, biases, dispatch="queue", **kw)
        for a, b in zip(out[:3], ref[:3]):
            assert torch.equal(a, b), rows is None
    g.close()


@pytest.mark.parametrize("direction", ["forward", "backward"])
def test_served_rows(direction):
    """One launch of requests of which some are filled first, and a launch of
    one request."""
    torch, tw = gpu_or_skip()
    g = _graph(torch, tw, False)
    reqs = [dict(num_walks=w, max_len=L, hop_bias=k, seed=i, direction=direction)
            for i, (w, L, k) in enumerate([(10, 5, "linear"), (700, 333, "uniform"),
                                           (0, 4000, "linear"), (64, 97, "linear"),
                                           (1, 100_001, "uniform"), (2000, 96, "linear")])]
    want = [g.sample_walks(dispatch="queue", **r) for r in reqs]
    srv = tw.Server(g, arena_bytes=64 << 20)
    for group in ([0, 1, 2, 3, 4, 5], [1], [4]):
        ids = [srv.submit(**reqs[i]) for i in group]
        for i, rid in zip(group, ids):
            for a, b in zip(srv.result(rid), want[i]):
                assert torch.equal(a, b), (group, i)
            srv.release(rid)
    srv.close()
    g.close()
