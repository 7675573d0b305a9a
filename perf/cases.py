"""Performance cases: the work that users of this library have it do, over the
ranges it is used in.

The graphs are the kinds the repository's benchmark and tests use, drawn on
the GPU from a seed: planted-partition SBM graphs (small and many-graph
workloads), R-MAT graphs (hubs, isolated vertices, merged weights) and
power-law graphs (the degree law of the headline's Chung-Lu graph, with
planted communities as crawled graphs have them).  Vertex counts need
not be powers of two.  A dynamic case applies one batch per pass: the batch,
then its inverse, then the batch again, so that the edge set stays in the
range of the case however often it runs (a sliding window inserts and
deletes in the same way).  Its state holds the planted communities, what a
static run recovers.

What each kind of call stands for:

* ``static``      communities of a graph that has just been loaded;
* ``df``          one update of a graph that is kept current (the batch edit
                  and Dynamic Frontier Louvain in one call);
* ``ds``          the same with Delta Screening, the serving loop's fallback;
* ``many``        one batch for each of many resident graphs in one launch
                  (a serving burst);
* ``modularity``  the quality of a labelling, as a monitor asks for it;
* ``static_f``, ``df_f``  the same calls in the paper's precision (float32
                  weights, FP64 sums).

ASYNC is the mode in use.  The reproducible SYNC mode is taken for static
runs on graphs without planted structure and for the state a dynamic case
on them starts from, since ASYNC results there differ from run to run.  An
ASYNC static pass names every community by its first vertex of a fixed
sample, as a program does that compares one clustering with the next.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2404_19634_amd import lib

DEV = "cuda"
GAMMA = 2.1             # degree exponent of the power-law graphs
HEAD = 64               # their heaviest vertices have weights of one order
RMAT = (0.57, 0.19, 0.19)
FLOAT_W = (0.25, 4.0)   # float32 weights of the paper-precision graphs


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def listed():
    return [
        # the smallest graphs: the 10,000-vertex planted-partition graph of the
        # tests and smoke run, loaded and then kept current; latency counts
        {"name": "static_sbm_10k", "kind": "static", "graph": "sbm", "n": 10_000, "block": 200, "mode": "async"},
        {"name": "df_sbm_10k_100", "kind": "df", "graph": "sbm", "n": 10_000, "block": 200, "updates": 100,
         "mode": "async"},
        # a graph with hubs and communities, loaded; ragged size
        {"name": "static_powerlaw_300k", "kind": "static", "graph": "powerlaw", "n": 300_007, "mode": "async"},
        # a graph with hubs and no clear communities, in the reproducible mode
        {"name": "static_rmat_700k_sync", "kind": "static", "graph": "rmat", "n": 700_001, "mode": "sync"},
        # updates of a graph with hubs: the benchmark's fractions 1e-5 and 1e-3
        {"name": "df_rmat_1m_160", "kind": "df", "graph": "rmat", "n": 1 << 20, "updates": 160, "mode": "async"},
        {"name": "df_rmat_1m_16000", "kind": "df", "graph": "rmat", "n": 1 << 20, "updates": 16_000, "mode": "async"},
        # the headline's degree law at a fifth of its size, with its large batch
        {"name": "df_powerlaw_4m_50000", "kind": "df", "graph": "powerlaw", "n": 4_000_000, "updates": 50_000,
         "mode": "async"},
        # the serving loop's fallback for a graph whose quality drifted
        {"name": "ds_sbm_300k_3000", "kind": "ds", "graph": "sbm", "n": 300_007, "block": 1500, "updates": 3_000,
         "mode": "async"},
        # a burst of the serving loop: 256 resident graphs, a 1e-3 |E| batch each
        {"name": "many_256", "kind": "many", "graphs": 256, "n_lo": 1_000, "n_hi": 50_000, "mode": "async"},
        # quality of a labelling of the benchmark's R-MAT graph
        {"name": "modularity_rmat_4m", "kind": "modularity", "graph": "rmat", "n": 1 << 22},
        # the paper's precision: a graph loaded, and a graph with hubs kept current
        {"name": "static_f_sbm_50k", "kind": "static_f", "graph": "sbm", "n": 50_003, "block": 500, "mode": "async"},
        {"name": "df_f_powerlaw_250k_1000", "kind": "df_f", "graph": "powerlaw", "n": 250_001, "updates": 1_000,
         "mode": "async"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["static", "df", "df", "ds", "many", "modularity", "static_f", "df_f"])
    if kind == "many":
        lo = _log(rng, 1_000, 4_000)
        return {"kind": kind, "graphs": _log(rng, 16, 256), "n_lo": lo, "n_hi": _log(rng, 2 * lo, 50_000),
                "mode": rng.choice(["async", "async", "sync"])}
    if kind == "modularity":
        return {"kind": kind, "graph": rng.choice(["rmat", "powerlaw"]), "n": _log(rng, 10_000, 2_000_000)}
    top = {"static": 300_000, "ds": 300_000, "static_f": 50_000, "df_f": 250_000, "df": 2_000_000}[kind]
    n = _log(rng, 10_000 if kind.startswith("static") else 5_000, top)
    if kind == "static":
        graph, mode = rng.choice([("sbm" if n < 60_000 else "powerlaw", "async"), ("powerlaw", "async"),
                                  ("rmat", "sync")])
    elif kind == "df":
        graph, mode = rng.choice([("sbm", "async"), ("powerlaw", "async"), ("powerlaw", "async"), ("rmat", "sync")])
    elif kind == "df_f":
        graph, mode = rng.choice(["sbm", "powerlaw"]), "async"
    else:
        graph, mode = "sbm", "async"
    case = {"kind": kind, "graph": graph, "n": n, "mode": mode}
    if graph == "sbm":  # blocks that the method resolves: at most about a hundred of them
        case["block"] = _log(rng, max(150, n // 100), max(200, n // 50))
    if kind in ("df", "ds", "df_f"):
        case["updates"] = _log(rng, 20, max(21, min(n // 50, 1_000 if kind == "df_f" else 50_000)))
    return case


# --------------------------------------------------------------------------
# inputs, drawn on the GPU from the seed
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2_654_435_761 % (1 << 62) + 17)
    return g


def _rand(k, g):
    return torch.rand(k, generator=g, device=DEV, dtype=torch.float64)


def _keys(a, b, n):
    ok = a != b
    a, b = a[ok], b[ok]
    return torch.minimum(a, b) * n + torch.maximum(a, b)


def _sbm_keys(n, gen, bstart, bsize, gstart, gsize):
    """Expected degree 24 inside the vertex's block and 4 in its graph: blocks
    that a static run finds whole, whatever the order of its moves."""
    def half(mean, start, size):
        a = (_rand(int(n * mean / 2), gen) * n).long()
        return a, start[a] + (_rand(a.numel(), gen) * size[a]).long()

    a, b = half(24, bstart, bsize)
    c, d = half(4, gstart, gsize)
    return torch.unique(_keys(torch.cat([a, c]), torch.cat([b, d]), n))


def _blocks(n, block):
    """Block index, first vertex and size of every vertex's block."""
    nb = max(1, n // block)
    v = torch.arange(n, device=DEV)
    lab = torch.clamp(v // block, max=nb - 1)
    size = torch.where(lab == nb - 1, n - block * (nb - 1), torch.full_like(lab, block))
    return lab, lab * block, size


def _edges(case, gen):
    """(u, v, w) of the case's graph: distinct pairs u < v, int32."""
    n, kind = case["n"], case["graph"]
    w = None
    if kind == "sbm":
        _, start, size = _blocks(n, case["block"])
        zero = torch.zeros_like(start)
        key = _sbm_keys(n, gen, start, size, zero, zero + n)
    elif kind == "rmat":
        m = 16 * n
        a = torch.zeros(m, dtype=torch.int64, device=DEV)
        b = torch.zeros_like(a)
        pa, pb, pc = RMAT
        for _ in range(max(1, (n - 1).bit_length())):
            r = torch.rand(m, generator=gen, device=DEV)
            low = r >= pa + pb
            right = ((r >= pa) & (r < pa + pb)) | (r >= pa + pb + pc)
            a = a * 2 + low
            b = b * 2 + right
        ok = (a < n) & (b < n)
        key, w = torch.unique(_keys(a[ok], b[ok], n), return_counts=True)
    else:  # powerlaw: mean degree 50 before merging, three quarters of it inside the vertex's community
        nb = _classes(n)
        a = _heavy(n, 25 * n, gen)
        inside = (a % nb) + nb * _heavy(n // nb, a.numel(), gen)
        b = torch.where(_rand(a.numel(), gen) < 0.75, inside, _heavy(n, a.numel(), gen))
        key, w = torch.unique(_keys(a, b, n), return_counts=True)
    if w is None:
        w = torch.ones_like(key)
    return key, w.int()


def _classes(n):
    """Planted communities of a power-law graph: vertex v is in v mod this."""
    return max(4, min(64, n // 2000))


def _heavy(n, k, gen):
    """k vertices below n, drawn with weight (v + HEAD)^(-1 / (GAMMA - 1))."""
    e = 1.0 - 1.0 / (GAMMA - 1.0)
    lo, hi = HEAD ** e, (n + HEAD) ** e
    return torch.clamp((lo + (hi - lo) * _rand(k, gen)).pow(1.0 / e) - HEAD, 0, n - 1).long()


def _split(key, n):
    return (key // n).int(), (key % n).int()


def _pick(m, k, gen):
    """k distinct indices below m, in random order."""
    idx = torch.unique((_rand(min(4 * m, k + k // 4 + 64), gen) * m).long())
    return idx[torch.argsort(_rand(idx.numel(), gen))[:k]]


def _batch(key, w, n, updates, gen, w_new):
    """80% insertions of absent pairs, 20% deletions of whole edges."""
    k_ins = max(1, int(round(0.8 * updates)))
    k_del = max(1, updates - k_ins)
    d = _pick(key.numel(), k_del, gen)
    c = k_ins + k_ins // 4 + 64
    new = torch.unique(_keys((_rand(c, gen) * n).long(), (_rand(c, gen) * n).long(), n))
    at = torch.clamp(torch.searchsorted(key, new), max=key.numel() - 1)
    new = new[key[at] != new]
    new = new[torch.argsort(_rand(new.numel(), gen))[:k_ins]]
    iu, iv = _split(new, n)
    flip = _rand(new.numel(), gen) < 0.5
    iu, iv = torch.where(flip, iv, iu), torch.where(flip, iu, iv)
    du, dv = _split(key[d], n)
    return (du, dv, w[d]), (iu, iv, w_new(new.numel(), gen))


def _unit(k, gen):
    return torch.ones(k, dtype=torch.int32, device=DEV)


def _float_w(k, gen):
    lo, hi = FLOAT_W
    return (lo + (hi - lo) * _rand(k, gen)).float()


def _both_ways(dels, ins, edges, batch):
    """The batch and its inverse."""
    return [batch(edges(*dels), edges(*ins)), batch(edges(*ins), edges(*dels))]


def _row_sums(n, u, v, w):
    """Weighted degrees: exact whole numbers, or float64 sums."""
    if w.dtype == torch.int32:
        def side(x, y):
            at = torch.searchsorted(x, torch.arange(n + 1, device=DEV, dtype=x.dtype))
            return torch.cat([y.new_zeros(1, dtype=torch.int64), y.cumsum(0)])[at].diff()

        order = torch.argsort(v)
        return side(u, w) + side(v[order], w[order])
    u, v, w = (x.cpu().numpy() for x in (u, v, w))
    k = np.bincount(u, weights=w, minlength=n) + np.bincount(v, weights=w, minlength=n)
    return torch.from_numpy(k).to(DEV)


def _planted(n, lab, k, cls):
    """The state of a labelling: what a program keeps after its static run."""
    c = lab.cpu().numpy()
    s = np.bincount(c, weights=k.cpu().numpy(), minlength=n)  # (whole numbers below 2^53 are exact)
    size = torch.from_numpy(np.bincount(c, minlength=n).astype(np.int32)).to(DEV)
    return cls(lab.int(), k, torch.from_numpy(s).to(DEV).to(k.dtype), size)


def _labels(n, gen):
    """Labels of a monitored clustering: community sizes spread widely."""
    c = max(2, int(math.sqrt(n)))
    return torch.clamp((c * _rand(n, gen) ** 3).int(), max=c - 1)


# --------------------------------------------------------------------------
# prepare
# --------------------------------------------------------------------------
def prepare(case, seed):
    kind, gen = case["kind"], _gen(seed)
    if kind == "many":
        return _prepare_many(case, gen)
    n = case["n"]
    real = kind.endswith("_f")
    key, w = _edges(case, gen)
    u, v = _split(key, n)
    if real:
        w = _float_w(key.numel(), gen)
        g = lib.GraphF.build(n, u, v, w, slack_frac=0.1, slack_min=8)
    else:
        g = lib.Graph.build(n, u, v, w, slack_frac=0.1, slack_min=8)
    s = {"kind": kind, "g": g, "flip": 0}
    if kind == "modularity":
        s["C"] = _labels(n, gen)
        return s
    s["prm"] = lib.params(mode=case["mode"])
    cls = lib.StateF if real else lib.State
    if kind.startswith("static"):
        s["state"] = cls.empty(n)
        s["ids"] = (torch.arange(0, n, max(1, n // 16_384), dtype=torch.int32, device=DEV)
                    if case["mode"] == "async" else None)
        return s
    if case["graph"] == "rmat":
        s["state"] = lib.louvain_static(g, mode="sync")[0]
    else:
        lab = (_blocks(n, case["block"])[0] if case["graph"] == "sbm"
               else torch.arange(n, device=DEV) % _classes(n))
        s["state"] = _planted(n, lab, _row_sums(n, u, v, w), cls)
    dels, ins = _batch(key, w, n, case["updates"], gen, _float_w if real else _unit)
    s["b"] = _both_ways(dels, ins, lib.EdgesF if real else lib.Edges, lib.BatchF if real else lib.Batch)
    return s


def _prepare_many(case, gen):
    count = case["graphs"]
    r = np.random.default_rng(case["graphs"] * 1_000_003 + case["n_lo"] * 31 + case["n_hi"])
    ns = np.exp(r.uniform(math.log(case["n_lo"]), math.log(case["n_hi"]), count)).astype(np.int64)
    bs = np.maximum(ns // r.integers(8, 60, count), 40)
    off = np.concatenate([[0], np.cumsum(ns)])
    total = int(off[-1])
    gi = torch.repeat_interleave(torch.arange(count, device=DEV), torch.from_numpy(ns).to(DEV))
    tn, tb, to = (torch.from_numpy(np.ascontiguousarray(x)).to(DEV) for x in (ns, bs, off[:-1]))
    local = torch.arange(total, device=DEV) - to[gi]
    nb = torch.clamp(tn // tb, min=1)[gi]
    lab = torch.minimum(local // tb[gi], nb - 1)
    size = torch.where(lab == nb - 1, tn[gi] - tb[gi] * (nb - 1), tb[gi])
    key = _sbm_keys(total, gen, to[gi] + lab * tb[gi], size, to[gi], tn[gi])
    w = torch.ones(key.numel(), dtype=torch.int32, device=DEV)
    u, v = _split(key, total)
    st = _planted(total, to[gi] + lab, _row_sums(total, u, v, w), lib.State)
    first = torch.searchsorted(key, torch.from_numpy(off).to(DEV) * total).tolist()
    s = {"kind": "many", "graphs": [], "states": [], "scratch": [], "max": [], "b": [[], []], "flip": 0,
         "prm": lib.params(mode=case["mode"]), "all": st}
    st.C.copy_(lab.int())
    need = 0
    for k in range(count):
        n, o = int(ns[k]), int(off[k])
        lo, hi = first[k], first[k + 1]
        lk = ((key[lo:hi] // total) - o) * n + (key[lo:hi] % total) - o
        lu, lv = _split(lk, n)
        g = lib.Graph.build(n, lu, lv, w[lo:hi], slack_frac=0.1, slack_min=8)
        need = max(need, g.workspace.numel())
        g._ws = None  # (one workspace serves the burst)
        s["graphs"].append(g)
        s["states"].append(lib.State(st.C[o:o + n], st.K[o:o + n], st.Sigma[o:o + n], st.size[o:o + n]))
        updates = max(5, (hi - lo) // 1000)
        dels, ins = _batch(lk, w[lo:hi], n, updates, gen, _unit)
        for side, b in enumerate(_both_ways(dels, ins, lib.Edges, lib.Batch)):
            s["b"][side].append(b)
        s["max"].append(updates + 8)
        s["scratch"].append(lib.many_scratch(n, updates + 8))
    s["ws"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    s["desc"] = torch.empty(int(lib.load().lv_many_desc_bytes(count)), dtype=torch.uint8, device=DEV)
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    kind, g = s["kind"], s.get("g")
    if kind == "modularity":
        return {"Q": lib.modularity(g, s["C"])}
    if kind == "static":
        return _named(lib.louvain_static(g, s["prm"], s["state"])[0], s["ids"])
    if kind == "static_f":
        return _named(lib.louvain_static_f(g, s["prm"], s["state"])[0], s["ids"])
    b = s["b"][s["flip"]]
    s["flip"] ^= 1
    if kind == "many":
        status, _ = lib.louvain_df_many(s["graphs"], b, s["states"], s["scratch"], s["max"], prm=s["prm"],
                                        ws=s["ws"], desc=s["desc"])
        return {"status": np.asarray(status), **_state(s["all"])}
    if kind == "df":
        lib.louvain_df_apply(g, b, s["state"], s["prm"])
    elif kind == "ds":
        lib.apply_batch(g, b)
        lib.louvain_ds(g, b, s["state"], s["prm"])
    else:
        lib.apply_batch_f(g, b)
        lib.louvain_df_f(g, b, s["state"], s["prm"])
    return {"row_len": g.row_len, "two_m": g.two_m_t, **_state(s["state"])}


def _state(st):
    return {"C": st.C, "K": st.K, "Sigma": st.Sigma, "size": st.size}


def _named(st, ids):
    """Per vertex: the first sampled vertex of its community, and the
    community's total and size."""
    if ids is None:
        return _state(st)
    c = st.C.long()
    first = torch.full_like(st.C, st.C.numel()).scatter_reduce_(0, c[ids], ids, "amin")
    return {"C": first[c], "K": st.K, "Sigma": st.Sigma[c], "size": st.size[c]}


# --------------------------------------------------------------------------
# what a pass cannot do without, and its floating outputs in 64 bits
# --------------------------------------------------------------------------
def work(case):
    """Static and modularity: every arc's neighbour and weight and the
    vertices' row bounds once, the results once.  Updates: the batch, and
    the rows of its endpoints with their neighbours' communities."""
    kind = case["kind"]
    if kind == "many":
        mean = (case["n_hi"] - case["n_lo"]) / math.log(case["n_hi"] / case["n_lo"])
        upd, deg = max(5.0, mean * 10 / 1000) * case["graphs"], 28
    else:
        deg = {"sbm": 28, "rmat": 32, "powerlaw": 40}[case["graph"]]
        arcs = case["n"] * deg
        if kind == "modularity":
            return {"bytes": 8 * arcs + 16 * case["n"], "flops": arcs}
        if kind.startswith("static"):
            return {"bytes": 8 * arcs + 12 * case["n"] + 24 * case["n"], "flops": 2 * arcs}
        upd = case["updates"]
        if kind == "ds":
            # (the screening's community flags send it over most communities' members)
            return {"bytes": 12 * upd + 12 * arcs + 24 * case["n"], "flops": 2 * arcs}
    return {"bytes": upd * (12 + 2 * (12 * deg + 36)), "flops": 4 * upd * deg}


def exact(case, seed):
    kind, gen = case["kind"], _gen(seed)
    if kind not in ("modularity", "static_f", "df_f"):
        return None  # whole numbers only
    n = case["n"]
    key, w = _edges(case, gen)
    u, v = _split(key, n)
    if kind == "modularity":
        c = _labels(n, gen).long()
        two_m = 2 * int(w.sum())
        intra = 2 * int(w[c[u.long()] == c[v.long()]].sum())
        tot = torch.zeros(n, dtype=torch.int64, device=DEV)
        tot.index_add_(0, c[u.long()], w.long()).index_add_(0, c[v.long()], w.long())
        return {"Q": (two_m * intra - int((tot * tot).sum())) / (two_m * two_m)}
    w = _float_w(key.numel(), gen)
    if kind == "static_f":
        return {"C": None, "K": _row_sums(n, u, v, w), "Sigma": None, "size": None}
    (du, dv, dw), (iu, iv, iw) = _batch(key, w, n, case["updates"], gen, _float_w)
    k = _row_sums(n, torch.cat([u, du, iu]), torch.cat([v, dv, iv]), torch.cat([w, -dw, iw]))
    two_m = 2 * (w.double().sum() - dw.double().sum() + iw.double().sum())
    return {"row_len": None, "two_m": two_m.reshape(1), "C": None, "K": k, "Sigma": None, "size": None}
