"""Rows written by walk blocks: every row width around their chunks of eight
slots, launches of one partial block to many, outputs that are not 16-byte
aligned, walks that never start; batches whose blocks take one bias each,
with given rows that do and do not cover the outputs. Against the queue
dispatch and the one-thread-per-walk batch, whose walks the oracle checks
elsewhere; equal bit for bit."""
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
def test_many_blocks(kind, direction):
    torch, tw = gpu_or_skip()
    if direction == "backward" and kind == "weight":
        pytest.skip("the weight-based picker walks forward only")
    g = _graph(torch, tw, directed=direction == "forward")
    for W, L in ((300_003, 9), (70_001, 8)):
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


@pytest.mark.parametrize("direction", ["forward", "backward"])
@pytest.mark.parametrize("W,L,base", [(1, 9, 0), (383, 12, 3), (385, 7, 2 ** 64 - 200),
                                      (100_003, 60, 5), (1_600_001, 9, 1)])
def test_batch_blocks(W, L, base, direction):
    """Six biases by walk id, uneven limits: rectangular rows, packed rows
    (above and below the size from which the rows are checked instead of
    pre-filled) and rows with gaps, which keep their padding."""
    torch, tw = gpu_or_skip()
    g = _graph(torch, tw, directed=direction == "forward")
    rng = np.random.default_rng(W)
    lim = torch.from_numpy(rng.integers(1, L + 1, W).astype(np.int32)).cuda()
    biases = [("uniform", 0.0, 1.0, 1.0), ("linear", 0.0, 1.0, 1.0), ("exponential", 300.0, 1.0, 1.0),
              ("node2vec", 300.0, 0.5, 2.0), ("node2vec", 300.0, 1.0, 1.0),
              ("node2vec", 300.0, 2.0, 0.5)]
    kw = dict(max_lens=lim, start_bias="linear", seed=3, walk_id_base=base, direction=direction)
    row, total = g.row_offsets(lim)
    gap = row + torch.arange(W + 1, device="cuda") // 2  # a free slot after every second row
    for rows in (None, (row, total), (gap, int(gap[-1]) + 3)):
        ragged = dict(ragged=True, rows=rows) if rows is not None else {}
        ref = g.sample_walks_batch(W, L, biases, dispatch="full_walk", **ragged, **kw)
        out = g.sample_walks_batch(W, L, biases, dispatch="queue", **ragged, **kw)
        for a, b in zip(out[:3], ref[:3]):
            assert torch.equal(a, b), (rows is None,)
    g.close()


def test_batch_bad_limits_and_rows():
    torch, tw = gpu_or_skip()
    g = _graph(torch, tw)
    W, L = 200_000, 30
    biases = [("uniform", 0.0, 1.0, 1.0), ("linear", 0.0, 1.0, 1.0)]
    lim = torch.full((W,), 30, dtype=torch.int32, device="cuda")
    row, total = g.row_offsets(lim)
    for where, bad in (("limit", 0), ("limit", 31), ("row", -1), ("row", W * 30 - 5)):
        l2, r2 = lim.clone(), row.clone()
        (l2 if where == "limit" else r2)[77] = bad
        for rows in (None, (r2, total)) if where == "limit" else ((r2, total),):
            ragged = dict(ragged=True, rows=rows) if rows is not None else {}
            nodes, ts, lens, _ = g.sample_walks_batch(W, L, biases, max_lens=l2, seed=1, **ragged)
            torch.cuda.synchronize()
            assert int(lens[77]) == 0 and int(lens[78]) >= 2
            assert bool((nodes.reshape(-1)[77 * 30:78 * 30] == -1).all())
            with pytest.raises(tw.TwError) as e:
                g.sync()
            assert e.value.code == tw.TW_EINVAL
    g.close()


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("start_mode", ["edge", "node"])
def test_hops_to_the_last_group(directed, start_mode):
    """Nodes of few groups, of one edge and of several, under a window that
    evicts down to one group and appends that join the last one: hops whose
    only candidate is the node's last group are answered from its record."""
    torch, tw = gpu_or_skip()
    rng = np.random.default_rng(11)
    V, W = 60, 20_000
    g = tw.Graph(V, directed=directed, window=8)
    t0 = 0
    for b in range(12):
        n = int(rng.integers(5, 120))
        ts = t0 + np.sort(rng.integers(0, 4, n)).astype(np.int64)
        t0 = int(ts[-1])  # the next batch may continue the last timestamp
        g.ingest_batch(*to_dev(torch, rng.integers(0, V, n).astype(np.int32),
                               rng.integers(0, V, n).astype(np.int32), ts))
        if b == 6:
            g.evict_before(t0)
        starts = torch.from_numpy(rng.integers(0, V, W).astype(np.int32)).cuda()
        for kind in ("uniform", "linear", "exponential", "node2vec", "weight"):
            kw = dict(hop_bias=kind, hop_tau=2.0, p=0.5, q=2.0, seed=b, start_mode=start_mode,
                      start_nodes=starts)
            ref = g.sample_walks(W, 8, dispatch="queue", **kw)
            for a, r in zip(g.sample_walks(W, 8, dispatch="full_walk", **kw), ref):
                assert torch.equal(a, r), (b, kind)
    g.close()


def test_rows_cut_short_by_the_outputs():
    """Rectangular rows over fewer slots than walks x width (out_slots of the
    C interface): walks whose limit still fits are written, the others are
    refused, and nothing is written past the last slot."""
    import ctypes

    torch, tw = gpu_or_skip()
    g = _graph(torch, tw)
    W, L, short = 500, 13, 500 * 13 - 6
    lim = torch.full((W,), 5, dtype=torch.int32, device="cuda")
    lim[W - 1] = 7
    lim[7] = 13
    starts = torch.zeros(W, dtype=torch.int32, device="cuda")

    def run(max_lens, slots):
        nodes = torch.full((W * L + 16,), 7, dtype=torch.int32, device="cuda")
        ts = torch.full((W * L + 16,), 7, dtype=torch.int64, device="cuda")
        lens = torch.full((W,), 7, dtype=torch.int32, device="cuda")
        biases = (tw._Bias * tw.MAX_BIASES)()
        for i in range(2):
            biases[i] = tw._Bias(i, 0.0, 1.0, 1.0)
        prm = tw._BatchParams(W, L, tw._ptr(max_lens), 2, biases, None, tw._Bias(0, 0.0, 1.0, 1.0),
                              tw.START_NODE, tw._ptr(starts), 3, 0, None, slots,
                              tw.DISPATCH["queue"], 0)
        tw._check(tw.lib().tw_sample_walks_batch(g._h, ctypes.byref(prm), tw._ptr(nodes),
                                                 tw._ptr(ts), tw._ptr(lens)))
        torch.cuda.synchronize()
        return nodes, ts, lens

    ref = run(lim, W * L)
    nodes, ts, lens = run(lim, short)  # the last row has 7 slots: its limit just fits
    g.sync()
    assert torch.equal(nodes[:short], ref[0][:short]) and torch.equal(ts[:short], ref[1][:short])
    assert torch.equal(lens, ref[2])
    assert bool((nodes[short:] == 7).all()) and bool((ts[short:] == 7).all())
    lim[W - 1] = 8
    nodes, ts, lens = run(lim, short)
    assert int(lens[W - 1]) == 0 and bool((nodes[short:] == 7).all())
    with pytest.raises(tw.TwError) as e:
        g.sync()
    assert e.value.code == tw.TW_EINVAL
    g.close()
