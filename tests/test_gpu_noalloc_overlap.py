"""Allocation-free calls that overlap: two graphs on two streams, no
synchronisation between their calls, and recorded calls replayed on both streams
at once. Every result equals the call's own, made alone."""
import numpy as np
import pytest

from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu

W, L = 40_000, 30


def _out(torch):
    return (torch.empty((W, L), dtype=torch.int32, device="cuda"),
            torch.empty((W, L), dtype=torch.int64, device="cuda"),
            torch.empty(W, dtype=torch.int32, device="cuda"))


def _call(g, i, out):
    kind = ["linear", "exponential", "uniform"][i % 3]
    g.sample_walks_noalloc(W, L, out, hop_bias=kind, hop_tau=300.0, seed=i, walk_id_base=i)


def test_overlapping_calls_and_replays():
    torch, tw = gpu_or_skip()
    streams = [torch.cuda.Stream() for _ in range(2)]
    graphs = []
    for k, s in enumerate(streams):
        rng = np.random.default_rng(20 + k)
        V, n = 2000, 200_000
        g = tw.Graph(V, stream=s)
        edges = to_dev(torch, rng.integers(0, V, n).astype(np.int32),
                       rng.integers(0, V, n).astype(np.int32),
                       np.sort(rng.integers(0, 30_000, n)).astype(np.int64))
        torch.cuda.synchronize()
        g.ingest_batch(*edges)
        graphs.append(g)
    want, got = [[[_out(torch) for _ in range(6)] for _ in graphs] for _ in range(2)]
    for k, g in enumerate(graphs):
        for i in range(6):
            _call(g, i, want[k][i])
            g.sync()

    def check():
        torch.cuda.synchronize()
        for k in range(2):
            for a, b in zip(got[k], want[k]):
                for x, y in zip(a, b):
                    assert torch.equal(x, y)
                    x.fill_(7)
        torch.cuda.synchronize()

    for i in range(6):
        for k, g in enumerate(graphs):
            _call(g, i, got[k][i])
    check()
    recorded = []
    for k, g in enumerate(graphs):
        r = torch.cuda.CUDAGraph()
        with torch.cuda.graph(r, stream=streams[k]):
            for i in range(6):
                _call(g, i, got[k][i])
        recorded.append(r)
    for _ in range(3):
        for k, r in enumerate(recorded):
            with torch.cuda.stream(streams[k]):
                r.replay()
        check()
    del recorded
    for g in graphs:
        g.close()
