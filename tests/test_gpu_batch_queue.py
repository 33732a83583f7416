"""The work queue of mixed batches. Biases that go by walk id run in walk blocks
under every dispatch but full_walk; given per walk they run on the queue, here
with the same biases given, so against the oracle's walks of the same ids: edge
and node starts, rectangular and packed rows, backward walks, a weight-based
bias among the others, any workgroups per compute unit."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import compare_walks, gpu_or_skip, to_dev
from test_gpu_batch import _mixed_graph, _oracle_batch

pytestmark = pytest.mark.gpu


def _unpack(nodes, ts, row, lims, L):
    W = len(lims)
    n = np.full((W, L), -1, np.int32)
    t = np.full((W, L), np.iinfo(np.int64).min, np.int64)
    for i in range(W):
        n[i, :lims[i]] = nodes[row[i]:row[i + 1]]
        t[i, :lims[i]] = ts[row[i]:row[i + 1]]
    return n, t


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("start_mode", ["edge", "node"])
@pytest.mark.parametrize("weight", [False, True])
def test_queue_forward(weight, start_mode, ragged):
    torch, tw = gpu_or_skip()
    g, og, tau = _mixed_graph(torch, tw)
    biases = synth.mixed_biases(tau)
    if weight:
        biases = biases[:4] + [("weight", tau, 1.0, 1.0)]
    W, L, seed, base = 12_000, 30, 7, 1000
    lims = synth.walk_lengths(3, W, 1, L)
    bidx = ((base + np.arange(W)) % len(biases)).astype(np.uint8)
    starts = synth.start_nodes(4, W, 3000)
    ref = _oracle_batch(og, W, L, biases, lims, bidx, seed, base, start_mode, starts)
    kw = dict(max_lens=to_dev(torch, lims)[0], bias_idx=to_dev(torch, bidx)[0], seed=seed,
              start_mode=start_mode, walk_id_base=base, ragged=ragged,
              start_nodes=to_dev(torch, starts)[0] if start_mode == "node" else None)
    for bpc in (0, 1):
        g.set_tuning(queue_bpc=bpc)
        nodes, ts, lens, row = g.sample_walks_batch(W, L, biases, **kw)
        g.sync()
        got = nodes.cpu().numpy(), ts.cpu().numpy()
        if ragged:
            got = _unpack(*got, row.cpu().numpy(), lims, L)
        _, boundary = compare_walks((*got, lens.cpu().numpy()), ref, exact=False)
        assert boundary <= max(2, W // 2000)
    g.close()


@pytest.mark.parametrize("directed", [True, False])
def test_queue_backward(directed):
    torch, tw = gpu_or_skip()
    V = 3000
    spec = synth.scaled("mixed", V, 40_000)["stream"]
    spec.directed = directed
    s, d, t = spec.all()
    g = tw.Graph(V, directed=directed)
    g.ingest_batch(*to_dev(torch, s, d, t))
    og = oracle.OracleGraph(V, directed=directed, backward=True)
    og.ingest_batch(s, d, t)
    tau = 0.1 * float(t.max() - t.min())
    biases = synth.mixed_biases(tau)
    W, L, seed, base = 12_000, 24, 17, 300
    lims = synth.walk_lengths(5, W, 1, L)
    bidx = ((base + np.arange(W)) % len(biases)).astype(np.uint8)
    nodes, ts, lens, _ = g.sample_walks_batch(
        W, L, biases, max_lens=to_dev(torch, lims)[0], bias_idx=to_dev(torch, bidx)[0], seed=seed,
        walk_id_base=base, direction="backward")
    g.sync()
    ref = _oracle_batch(og, W, L, biases, lims, bidx, seed, base, direction="backward")
    _, boundary = compare_walks((nodes.cpu().numpy(), ts.cpu().numpy(), lens.cpu().numpy()), ref,
                                exact=False)
    assert boundary <= max(2, W // 2000)
    g.close()
