"""Small batches (csrc/small.hip) and the sizes around their limit: one
workgroup's edit, updateWeights, marking and binning against the oracle, bit
for bit in SYNC mode."""
import numpy as np
import pytest

from paper_2404_19634_amd import workloads as W

pytestmark = pytest.mark.gpu


def _graph(n, seed):
    """Two hubs (rows beyond the workgroup bin), a ring, random weighted chords."""
    rng = np.random.default_rng(seed)
    p = {(0, v) for v in range(2, 4200)} | {(1, v) for v in range(1000, 3300)} | {(v, v + 1) for v in range(2, n - 1)}
    while len(p) < 3 * n:
        a, b = rng.integers(2, n, 2)
        if a != b:
            p.add((int(min(a, b)), int(max(a, b))))
    a = np.array(sorted(p), dtype=np.int32)
    return W.Edges(n, a[:, 0].copy(), a[:, 1].copy(), rng.integers(1, 4, len(a)).astype(np.int32))


def _batch(e, updates, seed):
    """A third deletions (many in the hub rows, some in part), the rest
    insertions: absent pairs, merges, and pairs the batch also deletes."""
    rng = np.random.default_rng(seed)
    nd = max(1, updates // 3)
    hub = np.nonzero(e.u == 0)[0]
    d = np.concatenate([rng.choice(hub, min(nd // 2, hub.size), replace=False),
                        rng.choice(np.nonzero(e.u > 1)[0], nd - min(nd // 2, hub.size), replace=False)])
    dw = np.where((np.arange(nd) % 3 == 0) & (e.w[d] > 1), e.w[d] - 1, e.w[d]).astype(np.int32)
    key = e.u.astype(np.int64) * e.n + e.v
    ni = updates - nd
    again = key[d[: min(nd, ni) // 4]]
    merge = rng.choice(key, min(ni // 4, 200), replace=False)
    a, b = rng.integers(2, e.n, 4 * updates + 8), rng.integers(2, e.n, 4 * updates + 8)
    new = (np.minimum(a, b) * e.n + np.maximum(a, b))[a != b]
    new = new[~np.isin(new, key)]
    pool = np.concatenate([again, merge, new])
    _, first = np.unique(pool, return_index=True)
    pick = pool[np.sort(first)][:ni]
    w = rng.integers(1, 5, pick.size).astype(np.int32)
    i32 = lambda x: np.ascontiguousarray(x.astype(np.int32))  # noqa: E731
    return W.Batch(i32(e.u[d]), i32(e.v[d]), dw, i32(pick % e.n), i32(pick // e.n), w)


@pytest.mark.parametrize("updates", [1, 2, 63, 255, 1023, 1024, 1025])
@pytest.mark.parametrize("n", [6001, 40_003])
@pytest.mark.parametrize("one_call", [True, False])
def test_sync_bit_exact(n, updates, one_call):
    import oracle
    from paper_2404_19634_amd import lib
    lib.set_tuning()
    e = _graph(n, n)
    b = _batch(e, updates, updates)
    assert b.size == updates
    g = lib.Graph.from_edges(e, slack_frac=0.5, slack_min=8)
    G = oracle.Graph.from_edges(e)
    st, _ = lib.louvain_static(g, mode="sync", max_iterations=6, max_passes=1)
    s0 = G.louvain("static", mode="sync", max_iterations=6, max_passes=1)[:3]
    d = lib.Batch.from_host(b)
    if one_call:
        st, gs = lib.louvain_df_apply(g, d, st, mode="sync")
    else:
        lib.apply_batch(g, d)
        st, gs = lib.louvain_df(g, d, st, mode="sync")
    assert G.apply_batch(b) == 0
    off, col, w = g.csr_host()
    o2, c2, w2 = G.csr()
    assert np.array_equal(off, o2) and np.array_equal(col, c2) and np.array_equal(w, w2)
    assert g.two_m == G.two_m
    Co, Ko, So, os_ = G.louvain("df", batch=b, state=s0, mode="sync")
    C, K, S = st.host()
    assert np.array_equal(C, Co) and np.array_equal(K, Ko) and np.array_equal(S, So)
    assert np.array_equal(st.size.cpu().numpy(), np.bincount(C, minlength=n))
    for k in ("passes", "iterations", "moves", "arcs_scanned", "vertices_affected", "iter_moves", "iter_gain"):
        assert gs[k] == os_[k], k


@pytest.mark.parametrize("updates", [1024, 1025])
@pytest.mark.parametrize("fault", ["id", "loop", "weight", "repeat", "missing", "heavy", "slack"])
def test_refused_batch_changes_nothing(updates, fault):
    from paper_2404_19634_amd import lib
    e = _graph(6001, 5)
    b = _batch(e, updates, 7)
    code = lib.LV_EINVAL
    if fault == "id":
        b.ins_u[-1] = 6001
    elif fault == "loop":
        b.ins_u[-1] = b.ins_v[-1]
    elif fault == "weight":
        b.ins_w[-1] = 0
    elif fault == "repeat":
        b.ins_u[-1], b.ins_v[-1] = b.ins_v[0], b.ins_u[0]
    elif fault == "missing":
        b.del_u[-1], b.del_v[-1] = 0, 1
        code = lib.LV_ENOEDGE
    elif fault == "heavy":
        b.del_w[-1] += 10
        code = lib.LV_ENOEDGE
    else:
        code = lib.LV_ENOSLACK
    g = lib.Graph.from_edges(e, slack_frac=0.0, slack_min=0 if fault == "slack" else 60)
    st, _ = lib.louvain_static(g, mode="sync", max_iterations=2, max_passes=1)
    before = [x.clone() for x in (g.row_len, g.col, g.w, g.two_m_t, st.C, st.K, st.Sigma, st.size)]
    for call in (lambda: lib.louvain_df_apply(g, lib.Batch.from_host(b), st), lambda: lib.apply_batch(g, lib.Batch.from_host(b))):
        with pytest.raises(lib.LouvainError) as ex:
            call()
        assert ex.value.code == code
        for x, y in zip(before, (g.row_len, g.col, g.w, g.two_m_t, st.C, st.K, st.Sigma, st.size)):
            assert bool((x == y).all())
