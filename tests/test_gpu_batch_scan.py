"""The batch edit's row scan: partners compared one by one (up to 16), looked
up by arc (rows of an arc per lane) or filtered.  One row of `length` arcs
loses and gains `partners` edges; the CSR matches the oracle's arc for arc."""
import numpy as np
import pytest

from paper_2404_19634_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [40, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025, 3000])
@pytest.mark.parametrize("partners", [1, 15, 16, 17, 38])
@pytest.mark.parametrize("others", [0, 1500])
def test_one_row(length, partners, others):
    import oracle
    from paper_2404_19634_amd import lib
    n = 6001
    rng = np.random.default_rng(length * 64 + partners)
    mates = np.sort(rng.choice(np.arange(1, 4000), length, replace=False))
    ring = np.arange(4000, n - 1)
    u = np.concatenate([np.zeros(length, np.int64), ring])
    v = np.concatenate([mates, ring + 1])
    w = rng.integers(2, 5, u.size)
    e = W.Edges(n, u.astype(np.int32), v.astype(np.int32), w.astype(np.int32))
    half = partners // 2
    d = rng.choice(length, half, replace=False)
    rest = np.setdiff1d(np.arange(length), d)
    merge = mates[rng.choice(rest, (partners - half) // 2, replace=False)]
    new = rng.choice(np.setdiff1d(np.arange(1, 4000), mates), partners - half - merge.size, replace=False)
    iu = np.concatenate([merge, new])
    dw = np.where(np.arange(half) % 2 == 0, w[d], 1)
    far = np.stack([np.arange(4000, 4000 + others), np.arange(4000, 4000 + others) + 2])  # (past the small path)
    b = W.Batch(np.zeros(half, np.int32), mates[d].astype(np.int32), dw.astype(np.int32),
                np.concatenate([np.zeros(iu.size), far[0]]).astype(np.int32),
                np.concatenate([iu, far[1]]).astype(np.int32), np.full(iu.size + others, 2, np.int32))
    g = lib.Graph.from_edges(e, slack_frac=1.0, slack_min=64)
    G = oracle.Graph.from_edges(e)
    lib.apply_batch(g, lib.Batch.from_host(b))
    assert G.apply_batch(b) == 0
    for x, y in zip(g.csr_host(), G.csr()):
        assert np.array_equal(x, y)
    assert g.two_m == 2 * (int(w.sum()) + 2 * (iu.size + others) - int(dw.sum()))
