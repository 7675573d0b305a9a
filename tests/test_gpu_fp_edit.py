"""The paper-precision batch edit against the FP oracle, arc for arc with
bit-equal float32 weights: by touched row (a small batch, hub rows in chunks
of 1024 arcs) and by pair (a batch of more updates than its scratch in the
pool has room for)."""
import numpy as np
import pytest

from paper_2404_19634_amd import workloads as W

pytestmark = pytest.mark.gpu


def _edges(n, pairs, seed):
    rng = np.random.default_rng(seed)
    a = np.array(sorted(pairs), dtype=np.int32)
    return W.Edges(n, a[:, 0].copy(), a[:, 1].copy(), rng.uniform(0.25, 4.0, len(a)).astype(np.float32))


def _hub(n, arcs):
    p = {(0, v) for v in range(1, arcs + 1)} | {(v, v + 1) for v in range(1, n - 1)}
    return _edges(n, p, arcs)


def _batch(e, n_del, ins, seed):
    """Whole and half deletions; insertions of absent and present pairs, and
    of pairs the batch also deletes (whole and half)."""
    rng = np.random.default_rng(seed)
    d = rng.choice(e.m, n_del, replace=False)
    dw = np.where(np.arange(n_del) % 2 == 0, e.w[d], e.w[d] * np.float32(0.5)).astype(np.float32)
    have = set(zip(e.u.tolist(), e.v.tolist()))
    pairs = {p for p in ins if p not in have}
    pairs |= {(int(e.u[k]), int(e.v[k])) for k in d[: n_del // 2]}
    pairs |= {(int(e.u[k]), int(e.v[k])) for k in rng.choice(e.m, n_del // 2, replace=False)}
    a = np.array(sorted(pairs), dtype=np.int32)
    iw = rng.uniform(0.25, 4.0, len(a)).astype(np.float32)
    return W.Batch(e.u[d], e.v[d], dw, a[:, 1].copy(), a[:, 0].copy(), iw)


@pytest.mark.parametrize("n,arcs", [(80, 63), (80, 64), (80, 65), (1100, 1023), (1100, 1025), (5000, 4097)])
def test_edit_by_row(n, arcs):
    import oracle
    from paper_2404_19634_amd import lib
    e = _hub(n, arcs)
    b = _batch(e, 20, [(2, n - 1), (0, n - 2), (5, n - 3)], n + arcs)
    _check(lib, oracle, e, b, slack_min=8)


@pytest.mark.parametrize("updates", [40, 1300])
def test_edit_of_a_small_graph(updates):
    import oracle
    from paper_2404_19634_amd import lib
    n, rng = 200, np.random.default_rng(updates)
    pairs = set()
    while len(pairs) < 1000:
        x, y = rng.integers(0, n, 2)
        if x != y:
            pairs.add((int(min(x, y)), int(max(x, y))))
    e = _edges(n, pairs, 4)
    ins = [(v, v + k) for v in range(n) for k in (91, 92, 93, 94, 95, 96, 97, 98)[: 1 + updates // 200] if v + k < n]
    _check(lib, oracle, e, _batch(e, min(600, updates // 2), ins, 3), slack_min=24)


def _check(lib, oracle, e, b, slack_min):
    g = lib.GraphF.build(e.n, e.u, e.v, e.w, slack_frac=0.0, slack_min=slack_min)
    G = oracle.GraphF.from_edges(e)
    before = g.two_m
    lib.apply_batch_f(g, lib.BatchF.from_host(b))
    G.apply_batch(b)
    off, col, w = g.csr_host()
    o2, c2, w2 = G.csr()
    assert np.array_equal(off, o2) and np.array_equal(col, c2)
    assert np.array_equal(w.view(np.uint32), w2.view(np.uint32))
    # 2m moves by the batch's weights in FP64 (the rows' float32 sums round)
    want = before + 2.0 * (b.ins_w.astype(np.float64).sum() - b.del_w.astype(np.float64).sum())
    assert abs(g.two_m - want) <= 1e-12 * want
