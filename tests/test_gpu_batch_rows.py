"""Row starts of a batch that no output can hold: near INT64_MAX the end of the
row, its start plus the walk's limit, does not fit 64 bits. Such a walk gets
length 0 and the call that synchronises next reports it; the others are as
without it. Walk blocks, the work queue (biases given per walk) and one thread
per walk."""
import numpy as np
import pytest

from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu

BIASES = [("uniform", 0.0, 1.0, 1.0), ("linear", 0.0, 1.0, 1.0)]


@pytest.mark.parametrize("form", ["blocks", "queue", "full_walk"])
@pytest.mark.parametrize("W,L", [(1000, 9), (200_000, 30)])
@pytest.mark.parametrize("start", [2 ** 63 - 1, 2 ** 63 - 5, -(2 ** 63), -1])
def test_row_starts_out_of_range(W, L, start, form):
    torch, tw = gpu_or_skip()
    rng = np.random.default_rng(5)
    V, n, at = 400, 6000, W - 40
    g = tw.Graph(V)
    g.ingest_batch(*to_dev(torch, rng.integers(0, V, n).astype(np.int32),
                           rng.integers(0, V, n).astype(np.int32),
                           rng.integers(0, 3000, n).astype(np.int64)))
    lim = torch.full((W,), L, dtype=torch.int32, device="cuda")
    row, total = g.row_offsets(lim)
    kw = dict(max_lens=lim, seed=2, ragged=True,
              dispatch="full_walk" if form == "full_walk" else "queue")
    if form == "queue":
        kw["bias_idx"] = (torch.arange(W, device="cuda") % 2).to(torch.uint8)
    want = g.sample_walks_batch(W, L, BIASES, rows=(row, total), **kw)
    bad = row.clone()
    bad[at] = start
    got = g.sample_walks_batch(W, L, BIASES, rows=(bad, total), **kw)
    torch.cuda.synchronize()
    with pytest.raises(tw.TwError) as e:
        g.sync()
    assert e.value.code == tw.TW_EINVAL
    for a, b, none in zip(got[:3], want[:3], (-1, tw.TS_NONE, 0)):
        b = b.clone()
        if b.numel() == W:
            b[at] = none
        else:
            b[at * L:(at + 1) * L] = none
        assert torch.equal(a, b)
    g.close()
