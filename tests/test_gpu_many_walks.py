"""More walks than a launch has threads (2^32): one batch and one served
request of rows of one slot. The lengths of all, and the walks around walk
2^32 and at the end, which a small call with those ids gives too."""
import numpy as np
import pytest

from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu

W, TAIL = 2 ** 32 + 100, 200


@pytest.mark.parametrize("path", ["batch", "serve"])
def test_more_walks_than_threads(path):
    torch, tw = gpu_or_skip()
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GiB of free device memory")
    rng = np.random.default_rng(7)
    V, n = 400, 6000
    g = tw.Graph(V)
    g.ingest_batch(*to_dev(torch, rng.integers(0, V, n).astype(np.int32),
                           rng.integers(0, V, n).astype(np.int32),
                           rng.integers(0, 3000, n).astype(np.int64)))
    want = g.sample_walks(TAIL, 1, seed=3, walk_id_base=W - TAIL)
    if path == "batch":
        nodes, ts, lens, _ = g.sample_walks_batch(W, 1, [("uniform", 0.0, 1.0, 1.0)], seed=3)
    else:
        srv = tw.Server(g, arena_bytes=65 << 30, hbm_reserve_bytes=-1)
        rid = srv.submit(num_walks=W, max_len=1, hop_bias="uniform", seed=3)
        assert srv.wait(rid)["status"] == tw.TW_OK
        nodes, ts, lens = srv.result(rid)
        srv.release(rid)
        srv.close()
    g.sync()
    for a, b in zip((nodes, ts, lens), want):
        assert torch.equal(a[-TAIL:], b)
    head = g.sample_walks(TAIL, 1, seed=3)
    for a, b in zip((nodes, ts, lens), head):
        assert torch.equal(a[:TAIL], b)
    for i in range(0, W, 1 << 30):
        assert bool((lens[i:i + (1 << 30)] == 1).all())
    del nodes, ts, lens
    torch.cuda.empty_cache()
    g.close()
