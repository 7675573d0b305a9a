"""Hub rows and large communities of the paper-precision path at the sizes
where the kernels change: the bins' edges (256, 2048 arcs), the LDS table of a
hub row (8192 slots, at most 6144 communities before the pool's table) and the
tiers of the aggregation (2048 arcs of members, 4096 communities of a level).
The weights are small multiples of 1/16, so every sum is exact in FP64 and the
expected moves hold exactly."""
import numpy as np
import pytest
import torch

from paper_2404_19634_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lib():
    from paper_2404_19634_amd import lib as L
    L.load()
    L.set_tuning()
    return L


def _star(D):
    # hub 0, leaves 1..D of one arc each (weight 1), leaf t with a mate D + 1
    t = 2 * D // 3 + 1
    u = np.zeros(D + 1, np.int32)
    v = np.arange(1, D + 2, dtype=np.int32)
    u[D] = t
    return t, W.Edges(D + 2, u, v, np.ones(D + 1, np.float32))


@pytest.mark.parametrize("with_size", [True, False])
@pytest.mark.parametrize("D", [255, 256, 257, 2047, 2048, 2049, 4096, 4097, 6143, 6144, 6145, 7200, 20000])
def test_hub_row_moves_to_its_best_community(lib, D, with_size):
    t, e = _star(D)
    n = e.n
    C = np.arange(n, dtype=np.int32)
    C[D + 1] = t
    K = np.bincount(e.u, minlength=n).astype(np.float64) + np.bincount(e.v, minlength=n)
    S = np.bincount(C, weights=K, minlength=n)
    g = lib.GraphF.build(n, e.u, e.v, e.w, slack_min=4)
    z, zf = np.zeros(0, np.int32), np.zeros(0, np.float32)
    b = W.Batch(z, z, zf, np.array([0], np.int32), np.array([t], np.int32), np.array([8.0], np.float32))
    bf = lib.BatchF.from_host(b)
    lib.apply_batch_f(g, bf)
    st = lib.StateF.from_host(C, K, S)
    if with_size:
        st.size = torch.from_numpy(np.bincount(C, minlength=n).astype(np.int32)).cuda()
    st, stats = lib.louvain_df_f(g, bf, st, max_iterations=1, max_passes=1)
    # t's community pays (9 - K_0 / m * 11 / 2) / m, every other one at most
    # 1 / m.  A longer row's bin runs before t's, which then is where it
    # belongs; up to 256 arcs both are in one launch, and t, which gains by
    # joining the hub too, may see it where it was.
    want = C.copy()
    want[0] = t
    got, K2, S2 = st.host()
    if D <= 256 and got[t] == 0:
        want[t] = 0
    assert np.array_equal(got, want)
    K[[0, t]] += 8.0
    assert np.array_equal(K2, K)
    assert np.array_equal(S2, np.bincount(want, weights=K, minlength=n))
    assert stats["moves"] == 1 + (got[t] == 0)


@pytest.mark.parametrize("pairs", [20, 700, 2047, 2048, 2300])
def test_aggregation_of_a_large_community(lib, pairs):
    """A heavy clique of 16 with one light arc to each of 2 x pairs triangles,
    which are joined by twos: the triangles are the first level's communities
    and the pairs the second's; the clique's super-vertex has 2 x pairs + 1
    neighbours."""
    core, tri = 16, 2 * pairs
    n = core + 3 * tri
    u, v, w = [], [], []
    for a in range(core):
        for c in range(a + 1, core):
            u.append(a), v.append(c), w.append(1024.0)
    base = core + 3 * np.arange(tri)
    for a, c in ((0, 1), (1, 2), (0, 2)):
        u.extend(base + a), v.extend(base + c), w.extend([1.0] * tri)
    u.extend(np.arange(tri) % core), v.extend(base), w.extend([0.5] * tri)
    u.extend(base[0::2] + 1), v.extend(base[1::2] + 1), w.extend([0.875] * pairs)
    g = lib.GraphF.build(n, np.array(u, np.int32), np.array(v, np.int32), np.array(w, np.float32))
    # (the clique holds most of the weight: the default tolerance would stop
    # before the triangles form)
    st, _ = lib.louvain_static_f(g, tolerance=1e-12, aggregation_tolerance=1.0)
    C, K, S = st.host()
    truth = np.concatenate([np.zeros(core, np.int64), 1 + np.arange(3 * tri) // 6])
    assert len(set(zip(C.tolist(), truth.tolist()))) == len(set(C.tolist())) == pairs + 1
    assert np.array_equal(S, np.bincount(C, weights=K, minlength=n))


def test_bad_membership_leaves_the_memberships(lib):
    _, e = _star(300)
    g = lib.GraphF.build(e.n, e.u, e.v, e.w, slack_min=4)
    st, _ = lib.louvain_static_f(g)
    before = st.C.clone()
    before[7] = e.n
    st.C.copy_(before)
    z, zf = np.zeros(0, np.int32), np.zeros(0, np.float32)
    b = W.Batch(z, z, zf, np.array([1], np.int32), np.array([2], np.int32), np.array([1.0], np.float32))
    with pytest.raises(lib.LouvainError) as ex:
        lib.louvain_df_f(g, lib.BatchF.from_host(b), st)
    assert ex.value.code == lib.LV_EINVAL
    assert torch.equal(st.C, before)
