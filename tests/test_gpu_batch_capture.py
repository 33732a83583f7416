"""A batch recorded in a HIP graph after a warm-up with another batch: any
batch call makes what a later one needs, so the recorded call allocates
nothing and its replays, with eager work in between, equal an eager call."""
import numpy as np
import pytest

from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu

BIASES = [("uniform", 0.0, 1.0, 1.0), ("linear", 0.0, 1.0, 1.0)]


@pytest.mark.parametrize("warm", ["blocks", "queue"])
@pytest.mark.parametrize("recorded", ["blocks", "queue"])
def test_large_ragged_batch_after_a_small_one(warm, recorded):
    torch, tw = gpu_or_skip()
    rng = np.random.default_rng(6)
    V, n, W, L = 400, 6000, 300_000, 30
    cap = torch.cuda.Stream()
    g = tw.Graph(V, stream=cap)
    edges = to_dev(torch, rng.integers(0, V, n).astype(np.int32),
                   rng.integers(0, V, n).astype(np.int32),
                   rng.integers(0, 3000, n).astype(np.int64))
    lim = torch.from_numpy(rng.integers(1, L + 1, W).astype(np.int32)).cuda()
    idx = torch.zeros(W, dtype=torch.uint8, device="cuda")  # biases per walk: the work queue
    torch.cuda.synchronize()
    g.ingest_batch(*edges)
    rows = g.row_offsets(lim)
    out, want = [(torch.empty(rows[1], dtype=torch.int32, device="cuda"),
                  torch.empty(rows[1], dtype=torch.int64, device="cuda"),
                  torch.empty(W, dtype=torch.int32, device="cuda")) for _ in range(2)]
    g.sample_walks_batch(100, 5, BIASES, bias_idx=idx if warm == "queue" else None)
    kw = dict(max_lens=lim, bias_idx=idx if recorded == "queue" else None, seed=5, ragged=True,
              rows=rows)
    held, layout = g.device_bytes(), g.walk_layout()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=cap):
        g.sample_walks_batch(W, L, BIASES, out=out, **kw)
    assert (g.device_bytes(), g.walk_layout()) == (held, layout)
    g.sample_walks_batch(W, L, BIASES, out=want, **kw)
    for _ in range(3):
        for x in out:
            x.fill_(7)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            assert torch.equal(a, b)
    del graph
    g.close()
