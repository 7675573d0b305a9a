"""The iteration plan (csrc/plan.hip): the frontier sorted by sub-round and
degree bin in one pass.  Vertex counts around multiples of the tile and the
32-vertex word; rows on both sides of every bin, class and hub boundary."""
import numpy as np
import pytest

from paper_2404_19634_amd import workloads as W

pytestmark = pytest.mark.gpu

ORDERS = [dict(), dict(async_round_order=0), dict(async_round_order=1), dict(async_rounds_log2=3),
          dict(revisit_min_degree=0), dict(revisit_min_degree=16), dict(revisit_min_degree=2000)]


@pytest.fixture
def lib():
    from paper_2404_19634_amd import lib as L
    L.load()
    L.set_tuning()
    yield L
    L.set_tuning()


def _graph(n, hubs):
    """A ring with `hubs` vertices whose row lengths sit at the boundaries."""
    want = [d for d in (4, 5, 8, 9, 16, 17, 32, 33, 128, 129, 256, 257, 1024, 1025, 2048, 2049, 4095, 4200) if d < n - 2]
    rng = np.random.default_rng(n)
    keys = {(v, v + 1) for v in range(n - 1)}
    for k in range(hubs):
        h = int(rng.integers(0, n))
        for v in rng.choice(n, want[k % len(want)], replace=False):
            if v != h:
                keys.add((min(h, int(v)), max(h, int(v))))
    a = np.array(sorted(keys), dtype=np.int32)
    return W.Edges(n, a[:, 0].copy(), a[:, 1].copy(), np.ones(a.shape[0], np.int32))


@pytest.mark.parametrize("n,hubs", [(63, 2), (4095, 9), (4096, 18), (4097, 36), (12_289, 54)])
def test_sync_bit_exact(lib, n, hubs):
    import oracle
    e = _graph(n, hubs)
    st, gs = lib.louvain_static(lib.Graph.from_edges(e), mode="sync", max_iterations=4)
    C, K, S = st.host()
    Co, Ko, So, os_ = oracle.Graph.from_edges(e).louvain("static", mode="sync", max_iterations=4)
    assert np.array_equal(C, Co) and np.array_equal(K, Ko) and np.array_equal(S, So)
    for k in ("iterations", "moves", "arcs_scanned", "vertices_affected", "iter_moves", "iter_gain"):
        assert gs[k] == os_[k], k


@pytest.mark.parametrize("order", ORDERS, ids=[str(o) or "default" for o in ORDERS])
@pytest.mark.parametrize("n,hubs", [(4096, 18), (12_289, 54)])
def test_async_visits_every_vertex_once_per_visit(lib, n, hubs, order):
    """One iteration over all vertices: each is in exactly one sub-round, and
    the classes above the revisit degree in one more."""
    lib.set_tuning(**order)
    e = _graph(n, hubs)
    deg = np.bincount(np.concatenate([e.u, e.v]), minlength=n)
    g = lib.Graph.from_edges(e)
    st, gs = lib.louvain_static(g, mode="async", max_iterations=1, max_passes=1)
    visits = np.ones(n, np.int64)
    if order.get("async_round_order", 2) == 2:
        rev = order.get("revisit_min_degree", 128)
        for lo, hi in ((1025, n), (129, 1024), (17, 128), (0, 16)):
            if rev > 0 and lo > rev:
                visits[(deg >= lo) & (deg <= hi)] = 2
    edges = (0, 4, 8, 16, 32, lib.get_tuning()["wave_max_degree"], 2048, n)
    for b in range(lib.NBINS):
        sel = (deg > edges[b]) & (deg <= edges[b + 1])
        assert gs["bin_vertices"][b] == int(visits[sel].sum()), b
        assert gs["bin_arcs"][b] == int((visits * deg)[sel].sum()), b
    assert gs["arcs_scanned"] == int((visits * deg).sum())
    assert gs["vertices_affected"] == n
    C, K, S = st.host()
    assert np.array_equal(K, deg)
    assert np.array_equal(S, np.bincount(C, weights=K, minlength=n).astype(np.int64))
    assert np.array_equal(st.size.cpu().numpy(), np.bincount(C, minlength=n))
