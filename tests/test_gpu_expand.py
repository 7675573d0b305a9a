"""The expansion of large iterations (pull or push by words, long rows, end)
and the launch that short rows share.  SYNC runs match the oracle bit for bit:
row lengths on both sides of a lane's 16 arcs, the push's 256 and the
workgroup's 2048, vertex counts around a wavefront's two words; a static run
whose row sums list long rows comes first in the workspace.  An ASYNC
iteration scans every row once whatever the wavefront's table."""
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


def _rows(n, degs, seed):
    """A ring plus vertices of the given row lengths."""
    rng = np.random.default_rng(seed)
    keys = {(v, v + 1) for v in range(n - 1)}
    for h, d in zip(rng.choice(n, len(degs), replace=False), degs):
        for v in rng.choice(n, min(d, n - 1), replace=False):
            if v != h:
                keys.add((min(int(h), int(v)), max(int(h), int(v))))
    a = np.array(sorted(keys), dtype=np.int32)
    return W.Edges(n, a[:, 0].copy(), a[:, 1].copy(), np.ones(a.shape[0], np.int32))


LENGTHS = (7, 8, 9, 15, 16, 17, 31, 48, 255, 256, 257, 2047, 2048, 2049, 5000)


@pytest.mark.parametrize("n", [2, 31, 32, 33, 63, 64, 65, 129, 6001, 20_031])
def test_sync_frontiers_match_the_oracle(lib, n):
    import oracle
    e = _rows(n, [d for d in LENGTHS if d < n], n)
    g, G = lib.Graph.from_edges(e), oracle.Graph.from_edges(e)
    for kw in (dict(), dict(max_iterations=3), dict(tolerance=0.0, max_iterations=12)):
        st, gs = lib.louvain_static(g, mode="sync", **kw)
        C, K, S = st.host()
        Co, Ko, So, os_ = G.louvain("static", mode="sync", **kw)
        assert np.array_equal(C, Co) and np.array_equal(K, Ko) and np.array_equal(S, So)
        for k in ("iterations", "moves", "arcs_scanned", "vertices_affected", "iter_moves", "iter_gain"):
            assert gs[k] == os_[k], (kw, k)
        assert abs(lib.modularity(g, st.C) - G.modularity(C)) <= 1e-12  # (shares the workspace)


@pytest.mark.parametrize("wave_max", [64, 128, 256, 512])
def test_async_short_rows_share_a_launch(lib, wave_max):
    lib.set_tuning(wave_max_degree=wave_max, revisit_min_degree=0)
    e = _rows(9001, LENGTHS[:-1] * 12, 5)
    g = lib.Graph.from_edges(e)
    st, gs = lib.louvain_static(g, mode="async", max_iterations=1, max_passes=1)
    deg = np.bincount(np.concatenate([e.u, e.v]), minlength=e.n)
    C, K, S = st.host()
    assert np.array_equal(K, deg) and np.array_equal(S, np.bincount(C, weights=deg, minlength=e.n).astype(np.int64))
    assert sum(gs["bin_vertices"]) >= e.n and gs["moves"] > 0
    assert gs["vertices_affected"] == e.n
