"""Modularity costs what its arcs cost, whatever share of them lies inside
communities."""
import time

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def skewed_graph(lib, n=2_000_000, classes=64, seed=1):
    """Rows of skewed length, three quarters of the arcs inside the classes
    v mod 64."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    r = lambda k: torch.rand(k, generator=g, device="cuda", dtype=torch.float64)  # noqa: E731
    m = 20 * n
    a = (n * r(m) ** 3).long()
    b = torch.where(r(m) < 0.75, a % classes + classes * ((n // classes) * r(m) ** 3).long(), (n * r(m) ** 3).long())
    ok = a != b
    a, b = a[ok], b[ok]
    key = torch.unique(torch.minimum(a, b) * n + torch.maximum(a, b))
    w = torch.ones(key.numel(), dtype=torch.int32, device="cuda")
    u, v = (key // n).int(), (key % n).int()
    return lib.Graph.build(n, u, v, w, slack_frac=0.1, slack_min=8), u, v


def median_time(lib, g, C, runs=15):
    ts = []
    for _ in range(runs + 3):
        torch.cuda.synchronize()
        t = time.perf_counter()
        q = lib.modularity(g, C)
        ts.append(time.perf_counter() - t)
    return float(np.median(ts[3:])), q


def test_good_labels_cost_what_random_ones_do():
    from paper_2404_19634_amd import lib
    g, u, v = skewed_graph(lib)
    planted = (torch.arange(g.n, device="cuda") % 64).int()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(2)
    random = planted[torch.randperm(g.n, generator=gen, device="cuda")]
    t_good, q_good = median_time(lib, g, planted)
    t_rand, q_rand = median_time(lib, g, random)
    assert q_good > 0.5 > q_rand
    assert t_good < 1.2 * t_rand, (t_good, t_rand)
