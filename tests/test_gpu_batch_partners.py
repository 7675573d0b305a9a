"""The batch edit's row scan on both sides of the partner counts where it
changes how it compares (4 for long rows, 16 for rows of an arc per lane)."""
import time

import numpy as np
import pytest
import torch

from tests.test_gpu_batch_scan import test_one_row as one_row

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [63, 64, 65, 66, 300, 1025, 1088, 1090])
@pytest.mark.parametrize("partners", [3, 4, 5, 6])
@pytest.mark.parametrize("others", [0, 1500])
def test_one_row(length, partners, others):
    one_row(length, partners, others)


def test_more_partners_cost_more():
    """Long rows that each get 16 partners (8192 updates of 1024 rows of
    20,000 arcs) are edited no slower than with 20 (10,240 updates)."""
    from paper_2404_19634_amd import lib
    H, deg = 1024, 20_000
    n = H + 4 * deg + 1000
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    h = torch.arange(H, device="cuda")
    leaf = torch.randint(H, n, (H * deg,), generator=gen, device="cuda")
    key = torch.unique(h.repeat_interleave(deg) * n + leaf)
    w = torch.ones(key.numel(), dtype=torch.int32, device="cuda")
    g = lib.Graph.build(n, (key // n).int(), (key % n).int(), w, slack_frac=0.1, slack_min=40)
    t = {}
    for partners in (16, 20):
        a = h.repeat(partners // 2)
        b = torch.cat([(h + d) % H for d in range(1, partners // 2 + 1)])
        e = lib.Edges(a.int(), b.int(), torch.ones(a.numel(), dtype=torch.int32, device="cuda"))
        none = lib.Edges([], [], [])
        ts = []
        for k in range(40):
            torch.cuda.synchronize()
            s = time.perf_counter()
            lib.apply_batch(g, lib.Batch(none, e) if k % 2 == 0 else lib.Batch(e, none))
            ts.append(time.perf_counter() - s)
        t[partners] = float(np.median(ts[4:]))
    assert t[16] < 1.05 * t[20], t
