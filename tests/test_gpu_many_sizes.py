"""The batched launch on both sides of the item count where it changes its
workgroup size, with rows around the 64-arc steps of a wavefront."""
import numpy as np
import pytest
import torch

from paper_2404_19634_amd import workloads as W

pytestmark = pytest.mark.gpu


def _graph(k):
    rng = np.random.default_rng(k)
    star = (0, 5, 63, 64, 65, 128, 129, 257)[k % 8]
    n = max(40, star + 3) + k % 7
    p = {(v, v + 1) for v in range(n - 1)} | {(0, v) for v in range(1, star + 1)}
    for _ in range(2 * n):
        a, b = rng.integers(0, n, 2)
        if a != b:
            p.add((int(min(a, b)), int(max(a, b))))
    a = np.array(sorted(p), dtype=np.int32)
    return W.Edges(n, a[:, 0].copy(), a[:, 1].copy(), rng.integers(1, 4, len(a)).astype(np.int32))


@pytest.mark.parametrize("count", [3, 512, 513])
def test_sync_bit_exact(count):
    import oracle
    from paper_2404_19634_amd import lib
    es = [_graph(k) for k in range(count)]
    bs = [W.random_batch(e, 9 + k % 23, k, ins_frac=0.6) for k, e in enumerate(es)]
    gs = [lib.Graph.from_edges(e, slack_frac=1.0, slack_min=8) for e in es]
    orc = [oracle.Graph.from_edges(e) for e in es]
    s0 = [G.louvain("static", mode="sync", max_iterations=3, max_passes=1)[:3] for G in orc]
    states = []
    for e, (C, K, S) in zip(es, s0):
        st = lib.State.from_host(C, K, S)
        st.size = torch.from_numpy(np.bincount(C, minlength=e.n).astype(np.int32)).cuda()
        states.append(st)
    scratch = [lib.many_scratch(e.n, 64) for e in es]
    ws = torch.empty(max(int(lib.load().lv_workspace_bytes(g.n, g.cap)) for g in gs), dtype=torch.uint8, device="cuda")
    status, stats = lib.louvain_df_many(gs, [lib.Batch.from_host(b) for b in bs], states, scratch, 64, ws=ws, mode="sync")
    assert status == [0] * count
    for k, (G, b) in enumerate(zip(orc, bs)):
        assert G.apply_batch(b) == 0
        Co, Ko, So, os_ = G.louvain("df", batch=b, state=s0[k], mode="sync")
        C, K, S = states[k].host()
        assert np.array_equal(C, Co) and np.array_equal(K, Ko) and np.array_equal(S, So), k
        assert stats[k]["moves"] == os_["moves"] and stats[k]["arcs_scanned"] == os_["arcs_scanned"], k
        if k % 16 == 0:
            off, col, w = gs[k].csr_host()
            o2, c2, w2 = G.csr()
            assert np.array_equal(off, o2) and np.array_equal(col, c2) and np.array_equal(w, w2), k
