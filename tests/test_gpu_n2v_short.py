"""node2vec walks of few nodes, whose lanes retry a rejected trial at once, and
the sizes on either side of that form: lengths 2 to 9, launches of 256, 1,600,
2,048 and 8,192 blocks and of one more, acceptance rates down to walks that end at the trial cap.
Against the queue dispatch, bit for bit."""
import numpy as np
import pytest

from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("direction", ["forward", "backward"])
@pytest.mark.parametrize("start_bias", ["uniform", "linear", "exponential"])
def test_short_node2vec_walks(start_bias, direction):
    torch, tw = gpu_or_skip()
    rng = np.random.default_rng(12)
    V, n = 300, 8000
    g = tw.Graph(V, directed=direction == "forward")
    g.ingest_batch(*to_dev(torch, rng.integers(0, V, n).astype(np.int32),
                           rng.integers(0, V, n).astype(np.int32),
                           np.sort(rng.integers(0, 3000, n)).astype(np.int64)))
    for W, lengths, pq in ((1, (4, 8), [(0.5, 2.0)]), (700, range(2, 10), [(0.5, 2.0), (2.0, 0.5)]),
                           (60, (3, 5, 8, 9), [(1e-7, 1.0), (1.0, 1e-3)]),
                           (16_384, (6, 8), [(2.0, 0.5)]), (16_385, (7, 8, 9), [(2.0, 0.5)]),
                           (102_401, (6, 8), [(2.0, 0.5)]), (131_072, (4, 6), [(2.0, 0.5)]),
                           (131_073, (4, 6), [(2.0, 0.5)]), (524_289, (4,), [(2.0, 0.5)])):
        for L in lengths:
            for p, q in pq:
                kw = dict(hop_bias="node2vec", hop_tau=300.0, p=p, q=q, start_bias=start_bias,
                          start_tau=300.0, seed=L, walk_id_base=9, direction=direction)
                ref = g.sample_walks(W, L, dispatch="queue", **kw)
                out = g.sample_walks(W, L, dispatch="full_walk", **kw)
                for a, b in zip(out, ref):
                    assert torch.equal(a, b), (W, L, p, q)
    g.close()
