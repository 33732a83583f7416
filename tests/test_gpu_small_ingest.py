"""Ingest at the sizes where its sorts and scans change form: the one-launch
sort (up to 4,096 records), the one-launch scans (up to 16,384 elements), 32-
and 64-bit sort keys, late drops of unsorted batches. Every view against the
oracle's."""
import numpy as np
import pytest

import oracle
from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("span", [40, 5000, 1 << 31, (1 << 32) + 5, 1 << 52])
@pytest.mark.parametrize("sizes", [(1, 2, 63, 64, 65, 255), (1023, 1024, 1025, 2047, 2048, 2049),
                                   (4095, 4096, 4097, 8191), (16383, 16384, 16385)])
def test_index_at_size_edges(directed, span, sizes):
    torch, tw = gpu_or_skip()
    rng = np.random.default_rng(sizes[0] + directed)
    V = 20_011
    g = tw.Graph(V, directed=directed, window=2 * span)
    og = oracle.OracleGraph(V, directed=directed, window=2 * span)
    t0 = -(1 << 40)
    for b, n in enumerate(sizes):
        src = (rng.zipf(1.5, n) % V).astype(np.int32)
        dst = rng.integers(0, V, n).astype(np.int32)
        ts = t0 + rng.integers(0, span, n).astype(np.int64)
        if b % 3 == 2:
            ts[: n // 4] -= 3 * span  # late records of an unsorted batch
        t0 += span // 2
        assert g.ingest_batch(*to_dev(torch, src, dst, ts)) == og.ingest_batch(src, dst, ts), b
        v, o = g.export_views(), og.views()
        for k in o:
            assert np.array_equal(v[k].cpu().numpy(), o[k]), (n, k)
    g.close()


def test_refused_id_in_any_workgroup():
    torch, tw = gpu_or_skip()
    n = 50_000
    for directed in (True, False):
        g = tw.Graph(100, directed=directed)
        src, dst, ts = to_dev(torch, np.zeros(n, np.int32), np.ones(n, np.int32),
                              np.arange(n, dtype=np.int64))
        for at, bad in ((0, 100), (n // 2, -1), (n - 1, 100)):
            s = src.clone()
            s[at] = bad
            with pytest.raises(tw.TwError) as e:
                g.ingest_batch(s, dst, ts)
            assert e.value.code == tw.TW_ERANGE
        assert g.ingest_batch(src, dst, ts)["accepted"] == n * (1 if directed else 2)
        g.close()
