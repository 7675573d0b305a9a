"""The iteration plan on both sides of one tile of 2048 vertices."""
import numpy as np
import pytest

from paper_2404_19634_amd import workloads as W
from tests.test_gpu_plan import _graph

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [31, 32, 33, 2047, 2048, 2049, 6143, 6145])
def test_sync_bit_exact(n):
    import oracle
    from paper_2404_19634_amd import lib
    lib.set_tuning()
    e = _graph(n, 7)
    st, gs = lib.louvain_static(lib.Graph.from_edges(e), mode="sync", max_iterations=4)
    C, K, S = st.host()
    Co, Ko, So, os_ = oracle.Graph.from_edges(e).louvain("static", mode="sync", max_iterations=4)
    assert np.array_equal(C, Co) and np.array_equal(K, Ko) and np.array_equal(S, So)
    for k in ("iterations", "moves", "arcs_scanned", "vertices_affected", "iter_moves", "iter_gain"):
        assert gs[k] == os_[k], k


@pytest.mark.parametrize("n", [2047, 2048, 2049])
def test_async_visits_every_vertex(n):
    from paper_2404_19634_amd import lib
    lib.set_tuning(revisit_min_degree=0)
    try:
        e = _graph(n, 9)
        g = lib.Graph.from_edges(e)
        st, gs = lib.louvain_static(g, mode="async", max_iterations=1, max_passes=1)
    finally:
        lib.set_tuning()
    deg = np.bincount(np.concatenate([e.u, e.v]), minlength=n)
    assert sum(gs["bin_vertices"]) == n and gs["vertices_affected"] == n
    assert gs["arcs_scanned"] == int(deg.sum())
    C, K, S = st.host()
    assert np.array_equal(K, deg)
    assert np.array_equal(S, np.bincount(C, weights=K, minlength=n).astype(np.int64))
