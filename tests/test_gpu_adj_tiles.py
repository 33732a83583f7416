"""node2vec's pair table counted in tiles of 4 and of 16 records a thread (from
786,432 records up and down together): built over a window of either size, kept
current by batches of either size with few distinct pairs, whose records repeat
within a tile and over tiles. Walks against the oracle's."""
import numpy as np
import pytest

import oracle
from gpu_util import compare_walks, gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(786_431, 786_433, 500), (300_000, 450_000, 450_000, 300_000)])
def test_pair_table(sizes):
    torch, tw = gpu_or_skip()
    rng = np.random.default_rng(len(sizes))
    V, window, W = 120, 15_000, 4000
    g = tw.Graph(V, window=window)
    og = oracle.OracleGraph(V, window=window)
    for b, n in enumerate(sizes):
        e = ((rng.zipf(1.3, n) % V).astype(np.int32), (rng.zipf(1.3, n) % V).astype(np.int32),
             (10_000 * b + np.sort(rng.integers(0, 10_000, n))).astype(np.int64))
        assert g.ingest_batch(*to_dev(torch, *e)) == og.ingest_batch(*e)
        kw = dict(hop_bias="node2vec", hop_tau=1500.0, p=0.25, q=4.0, seed=b)
        out = g.sample_walks(W, 12, **kw)
        g.sync()
        ref = og.sample_walks(W, 12, with_margin=True, **kw)
        _, boundary = compare_walks(tuple(x.cpu().numpy() for x in out), ref, exact=False)
        assert boundary <= 4
    g.close()
