"""Small batches whose endpoints are hub rows: the pool slots and units that
the one-workgroup start hands out (csrc/small.hip), against the oracle, bit
for bit in SYNC mode."""
import numpy as np
import pytest

from paper_2404_19634_amd import workloads as W

pytestmark = pytest.mark.gpu

LENGTHS = (2049, 2050, 4095, 4097, 2048, 2303, 8193)  # (2048: not a hub row)


def _hub_graph(hubs, seed):
    """`hubs` vertices with rows of the lengths above over one ring of leaves."""
    rng = np.random.default_rng(seed)
    n = hubs + 9001
    key = [np.arange(hubs, n - 1, dtype=np.int64) * n + np.arange(hubs + 1, n)]
    for h in range(hubs):
        v = hubs + rng.permutation(n - hubs)[: LENGTHS[h % len(LENGTHS)]]
        key.append(h * np.int64(n) + v)
    k = np.concatenate(key)
    w = rng.integers(1, 4, k.size).astype(np.int32)
    return W.Edges(n, (k // n).astype(np.int32), (k % n).astype(np.int32), w)


def _hub_batch(hubs, updates, seed):
    """Distinct pairs of hubs, every hub in one of the first hubs/2 pairs."""
    rng = np.random.default_rng(seed)
    p = rng.permutation(hubs)
    pairs = {tuple(sorted((int(p[2 * k]), int(p[2 * k + 1])))) for k in range(hubs // 2)}
    assert len(pairs) <= updates
    while len(pairs) < updates:
        a, b = rng.integers(0, hubs, 2)
        if a != b:
            pairs.add((int(min(a, b)), int(max(a, b))))
    a = np.array(sorted(pairs), dtype=np.int32)
    none = np.zeros(0, np.int32)
    return W.Batch(none, none, none, a[:, 0].copy(), a[:, 1].copy(), rng.integers(1, 5, updates).astype(np.int32))


@pytest.mark.parametrize("hubs,updates", [(2, 1), (3, 3), (64, 300), (1024, 513), (1027, 1024), (1350, 1024)])
def test_sync_bit_exact(hubs, updates):
    import oracle
    from paper_2404_19634_amd import lib
    lib.set_tuning()
    e = _hub_graph(hubs, hubs)
    b = _hub_batch(hubs, updates, updates)
    g = lib.Graph.from_edges(e, slack_frac=0.02, slack_min=16)
    G = oracle.Graph.from_edges(e)
    k0 = np.bincount(e.u, weights=e.w, minlength=e.n) + np.bincount(e.v, weights=e.w, minlength=e.n)
    C0 = np.arange(e.n, dtype=np.int32)  # (singletons: every update marks both ends)
    k0 = k0.astype(np.int64)
    st = lib.State.from_host(C0, k0, k0)
    st, gs = lib.louvain_df_apply(g, lib.Batch.from_host(b), st, mode="sync", max_iterations=2, max_passes=1)
    assert G.apply_batch(b) == 0
    Co, Ko, So, os_ = G.louvain("df", batch=b, state=(C0, k0, k0), mode="sync", max_iterations=2, max_passes=1)
    C, K, S = st.host()
    assert np.array_equal(C, Co) and np.array_equal(K, Ko) and np.array_equal(S, So)
    for k in ("iterations", "moves", "arcs_scanned", "vertices_affected", "iter_moves", "iter_gain"):
        assert gs[k] == os_[k], k
    if updates >= hubs // 2:
        assert gs["bin_vertices"][lib.BINS.index("hub")] > 0
