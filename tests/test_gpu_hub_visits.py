"""Hub rows in planned ASYNC iterations: a second visit starts from clean
sums, and rows above 2^20 arcs use cleared tables, one sub-round after
another and from the small-batch start."""
import numpy as np
import pytest

from paper_2404_19634_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture
def lib():
    from paper_2404_19634_amd import lib as L
    L.load()
    L.set_tuning()
    yield L
    L.set_tuning()


def _second_visit(p, q, s, r):
    """Vertices h and g (the first two of the order below), p leaves of h in
    community A, q leaves of h and r leaves of g in community B, an arc h-g of
    weight s, h and g in A, and a far pair whose weight outweighs every total.
    The degree class of h and g is visited twice, h's sub-round before g's.
    First visit: h has p + s into A and q < p + s into B and stays; g has s into
    A and r > s into B and leaves.  Second visit: p into A, q + s > p into B, so
    h follows.  With the first visit's sum still in it, A would hold it:
    2 p + s > q + s."""
    n = 2 + p + q + r + 2
    rnd = (np.arange(n, dtype=np.uint32) * np.uint32(0x9E3779B1)) >> np.uint32(27)
    h = int(np.nonzero(rnd == 3)[0][0])
    g = int(np.nonzero(rnd == 20)[0][0])
    rest = np.setdiff1d(np.arange(n), [h, g])
    la, lb, lg, far = np.split(rest, np.cumsum([p, q, r]))
    u = np.concatenate([np.full(p + q, h), np.full(r, g), [h], far[:1]])
    v = np.concatenate([la, lb, lg, [g], far[1:]])
    w = np.concatenate([np.ones(p + q + r, np.int64), [s, 9 * 10**8]])
    e = W.Edges(n, u.astype(np.int32), v.astype(np.int32), w.astype(np.int32))
    A, B = int(la[0]), int(lb[0])
    C = np.empty(n, np.int32)
    C[la] = C[h] = C[g] = A
    C[lb] = C[lg] = B
    C[far] = far[0]
    want = np.full(n, B, np.int32)  # every leaf then follows its hub
    want[far] = far[0]
    return e, C, want, h, g


@pytest.mark.parametrize("p,q,s,r", [(1000, 1200, 300, 1300), (2900, 3000, 300, 2100),
                                     (500_000, 600_000, 150_000, 1_100_000)])
def test_async_hub_moves_on_its_second_visit(lib, p, q, s, r):
    e, C, want, h, g = _second_visit(p, q, s, r)
    n = e.n
    K = (np.bincount(e.u, weights=e.w, minlength=n) + np.bincount(e.v, weights=e.w, minlength=n)).astype(np.int64)
    S = np.bincount(C, weights=K, minlength=n).astype(np.int64)
    st = lib.State.from_host(C, K, S)
    none = lib.Edges([], [], [])
    gr = lib.Graph.from_edges(e)
    st, t = lib.louvain_nd(gr, lib.Batch(none, none), st, mode="async", max_iterations=1, max_passes=1)
    Cg, Kg, Sg = st.host()
    assert Cg[h] == want[h] and Cg[g] == want[g]
    assert np.array_equal(Cg, want) and np.array_equal(Kg, K)
    assert np.array_equal(Sg, np.bincount(want, weights=K, minlength=n).astype(np.int64))
    assert t["bin_vertices"][lib.BINS.index("hub")] == 2 * (1 + (r > 2047))
    assert t["moves"] == 2 + p


@pytest.mark.parametrize("one_call", [True, False])
def test_small_batch_on_a_row_above_2_20_arcs(lib, one_call):
    """The one-workgroup start leaves such a row's table to be cleared."""
    import oracle
    leaves, n = (1 << 20) + 70, (1 << 20) + 80
    i32 = lambda *x: np.array(x, np.int32)  # noqa: E731
    u = np.concatenate([np.zeros(leaves, np.int32), np.arange(1, n - 1, dtype=np.int32)])
    v = np.concatenate([np.arange(1, leaves + 1, dtype=np.int32), np.arange(2, n, dtype=np.int32)])
    e = W.Edges(n, u, v, np.ones(u.size, np.int32))
    k = np.bincount(np.concatenate([u, v]), minlength=n).astype(np.int64)
    rng = np.random.default_rng(5)
    # 40 communities, so that the row's segments hold sums of many arcs
    C0 = rng.integers(0, 40, n).astype(np.int32)
    S0 = np.bincount(C0, weights=k, minlength=n).astype(np.int64)
    b = W.Batch(i32(), i32(), i32(), i32(0, 0, 5), i32(leaves + 2, leaves + 5, 900), i32(1, 2, 1))
    G = oracle.Graph.from_edges(e)
    assert G.apply_batch(b) == 0
    g = lib.Graph.from_edges(e)
    d = lib.Batch.from_host(b)
    for _ in range(2):  # (the second run finds the first one's table in the workspace)
        st = lib.State.from_host(C0, k, S0)
        if one_call and _ == 0:
            st, gs = lib.louvain_df_apply(g, d, st, mode="sync", max_iterations=2, max_passes=1)
        else:
            if _ == 0:
                lib.apply_batch(g, d)
            st, gs = lib.louvain_df(g, d, st, mode="sync", max_iterations=2, max_passes=1)
        Co, Ko, So, os_ = G.louvain("df", batch=b, state=(C0, k, S0), mode="sync", max_iterations=2, max_passes=1)
        C, K, S = st.host()
        assert np.array_equal(C, Co) and np.array_equal(K, Ko) and np.array_equal(S, So)
        for key in ("iterations", "moves", "arcs_scanned", "vertices_affected", "iter_moves", "iter_gain"):
            assert gs[key] == os_[key], key
        assert gs["bin_vertices"][lib.BINS.index("hub")] > 0
