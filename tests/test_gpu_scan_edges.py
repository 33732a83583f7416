"""Scans at the sizes where they change form, one workgroup with its elements a
thread or two launches: 7,168 for 64-bit sums, 12,288 for 32-bit ones (an
ingest's, whose index is checked against the oracle's)."""
import numpy as np
import pytest

import oracle
from gpu_util import gpu_or_skip, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [0, 1, 63, 1023, 1024, 1025, 6145, 7167, 7168, 7169, 8192, 16_385])
def test_row_offsets(n):
    torch, tw = gpu_or_skip()
    g = tw.Graph(10)
    gen = torch.Generator(device="cuda").manual_seed(n)
    x = torch.randint(0, 1 << 30, (n,), generator=gen, device="cuda").int()
    row, total = g.row_offsets(x)
    want = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), x.long().cumsum(0)])
    assert torch.equal(row, want) and total == int(want[-1])
    g.close()


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("n", [6143, 6144, 6145, 12_287, 12_288, 12_289])
def test_ingest(n, directed):
    torch, tw = gpu_or_skip()
    rng = np.random.default_rng(n)
    V = 40_000  # about as many nodes touched as records
    g = tw.Graph(V, directed=directed, window=5000)
    og = oracle.OracleGraph(V, directed=directed, window=5000)
    for b in range(3):
        e = (rng.permutation(V)[:n].astype(np.int32), rng.permutation(V)[:n].astype(np.int32),
             (3000 * b + rng.integers(0, 3000, n)).astype(np.int64))
        assert g.ingest_batch(*to_dev(torch, *e)) == og.ingest_batch(*e)
        v, o = g.export_views(), og.views()
        for k in o:
            assert np.array_equal(v[k].cpu().numpy(), o[k]), k
    g.close()
