"""tw_server_copy_out into memory that is not the graph's device's own: pinned
host memory, and (with two devices) another GPU's, which the copy has to reach
without the caller enabling peer access. Equal to the plain walks."""
import ctypes

import numpy as np
import pytest

from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


def _outputs(torch, W, L, where):
    kw = dict(pin_memory=True) if where == "pinned" else dict(device=where)
    return (torch.empty((W, L), dtype=torch.int32, **kw), torch.empty((W, L), dtype=torch.int64, **kw),
            torch.empty(W, dtype=torch.int32, **kw))


@pytest.mark.parametrize("where", ["cuda:0", "pinned", "cuda:1"])
def test_copy_out_destinations(where):
    torch, tw = gpu_or_skip()
    if where == "cuda:1" and torch.cuda.device_count() < 2:
        pytest.skip("one GPU")
    rng = np.random.default_rng(4)
    V, n, W, L = 300, 5000, 777, 13
    g = tw.Graph(V)
    g.ingest_batch(*to_dev(torch, rng.integers(0, V, n).astype(np.int32),
                           rng.integers(0, V, n).astype(np.int32),
                           np.sort(rng.integers(0, 3000, n)).astype(np.int64)))
    want = g.sample_walks(W, L, hop_bias="linear", seed=8)
    srv = tw.Server(g, arena_bytes=16 << 20)
    rid = srv.submit(num_walks=W, max_len=L, hop_bias="linear", seed=8)
    assert srv.wait(rid)["status"] == tw.TW_OK
    out = _outputs(torch, W, L, where)
    tw._check(tw.lib().tw_server_copy_out(srv._h, ctypes.c_uint64(rid),
                                          *(ctypes.c_void_p(x.data_ptr()) for x in out)))
    for a, b in zip(out, want):
        assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())
    srv.release(rid)
    srv.close()
    g.close()
