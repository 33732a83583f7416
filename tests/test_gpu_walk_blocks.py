"""Rows written by the full-walk kernel's blocks: every row width around its
chunks of four and eight slots, launches of one partial block to several
rounds a wavefront, outputs that are not 16-byte aligned, walks that never
start. Against the queue dispatch, whose walks the oracle checks elsewhere;
equal bit for bit."""
import numpy as np
import pytest

from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


def _graph(torch, tw, V=400, n=6000, directed=True):
    rng = np.random.default_rng(3)
    g = tw.Graph(V, directed=directed)
    g.ingest_batch(*to_dev(torch, rng.integers(0, V - 3, n).astype(np.int32),
                           rng.integers(0, V, n).astype(np.int32),
                           rng.integers(0, 3000, n).astype(np.int64)))
    return g


def _outputs(torch, W, L, shift):
    """(nodes, ts, len) with the row arrays starting `shift` slots past an
    aligned address, between guard slots."""
    n = torch.full((W * L + 16,), 7, dtype=torch.int32, device="cuda")
    t = torch.full((W * L + 16,), 7, dtype=torch.int64, device="cuda")
    return n, t, (n[shift:shift + W * L].view(W, L), t[shift:shift + W * L].view(W, L),
                  torch.full((W,), 7, dtype=torch.int32, device="cuda"))


@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 7, 8, 9, 12, 25, 4100])
@pytest.mark.parametrize("shift", [0, 1, 4])
@pytest.mark.parametrize("kind", ["uniform", "node2vec"])
def test_rows_of_any_width(L, shift, kind):
    torch, tw = gpu_or_skip()
    g = _graph(torch, tw)
    for W in (1, 63, 64, 65, 1000) if L < 100 else (65,):
        rng = np.random.default_rng(W)
        starts = torch.from_numpy(rng.integers(0, 400, W).astype(np.int32)).cuda()
        kw = dict(hop_bias=kind, hop_tau=300.0, p=0.5, q=2.0, start_mode="node",
                  start_nodes=starts, seed=W, walk_id_base=5)
        ref = g.sample_walks(W, L, dispatch="queue", **kw)
        n, t, out = _outputs(torch, W, L, shift)
        g.sample_walks(W, L, dispatch="full_walk", out=out, **kw)
        g.sync()
        for a, b in zip(out, ref):
            assert torch.equal(a, b), (W, L)
        for x in (n, t):  # nothing outside the rows
            assert bool((x[:shift] == 7).all()) and bool((x[shift + W * L:] == 7).all())
    g.close()


@pytest.mark.parametrize("kind", ["uniform", "linear", "exponential", "node2vec", "weight"])
@pytest.mark.parametrize("direction", ["forward", "backward"])
def test_several_rounds_a_wavefront(kind, direction):
    torch, tw = gpu_or_skip()
    if direction == "backward" and kind == "weight":
        pytest.skip("the weight-based picker walks forward only")
    g = _graph(torch, tw, directed=direction == "forward")
    for W, L in ((1_100_003, 9), (700_001, 8)):
        kw = dict(hop_bias=kind, hop_tau=300.0, p=2.0, q=0.5, start_bias="linear", seed=L,
                  direction=direction)
        ref = g.sample_walks(W, L, dispatch="queue", **kw)
        out = g.sample_walks(W, L, dispatch="full_walk", **kw)
        for a, b in zip(out, ref):
            assert torch.equal(a, b), (W, L)
    g.close()


def test_bad_start_nodes_leave_padded_rows():
    torch, tw = gpu_or_skip()
    g = _graph(torch, tw)
    W, L = 300, 6
    starts = torch.arange(W, dtype=torch.int32, device="cuda")
    starts[::3] = 400
    starts[1::3] = 399  # a node without edges
    nodes, ts, lens = g.sample_walks(W, L, start_mode="node", start_nodes=starts,
                                     dispatch="full_walk")
    torch.cuda.synchronize()
    assert bool((lens[::3] == 0).all()) and bool((nodes[::3] == -1).all())
    assert bool((lens[1::3] == 1).all()) and bool((nodes[1::3, 1:] == -1).all())
    assert bool((ts[::3] == tw.TS_NONE).all()) and bool((ts[1::3] == tw.TS_NONE).all())
    with pytest.raises(tw.TwError) as e:
        g.sync()
    assert e.value.code == tw.TW_ERANGE
    g.close()
