"""Modularity on graphs around the size where one-byte label tags filter the
gathers of C, with labels whose tags collide and rows on both sides of every
row-sum class."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1 << 20, (1 << 20) + 1, (1 << 20) + 3])
@pytest.mark.parametrize("labels", ["few", "same_tag", "many"])
def test_label_tags(n, labels):
    from paper_2404_19634_amd import lib
    rng = np.random.default_rng(n)
    u = [np.arange(n - 1, dtype=np.int64)]
    v = [np.arange(1, n, dtype=np.int64)]
    for h, deg in enumerate((3, 4, 14, 15, 62, 63, 64, 4094, 4095, 9000)):
        t = rng.choice(np.arange(100, n, dtype=np.int64), deg, replace=False)
        u.append(np.full(deg, 3 * h))
        v.append(t)
    u, v = np.concatenate(u), np.concatenate(v)
    w = rng.integers(1, 5, u.size)
    if labels == "few":
        c = rng.integers(0, 3, n)
    elif labels == "same_tag":  # different labels with one tag
        x = np.arange(n, dtype=np.uint64)
        tag = ((x * np.uint64(0x9E3779B1)) & np.uint64(0xFFFFFFFF)) >> np.uint64(24)
        c = rng.choice(np.nonzero(tag == 7)[0][:5], n)
    else:
        c = np.arange(n) // 3
    g = lib.Graph.build(n, u, v, w)
    q = lib.modularity(g, torch.from_numpy(c.astype(np.int32)).cuda())
    two_m = 2 * int(w.sum())
    tot = np.bincount(c[u], weights=w, minlength=n) + np.bincount(c[v], weights=w, minlength=n)
    num = two_m * 2 * int(w[c[u] == c[v]].sum()) - int((tot.astype(np.int64) ** 2).sum())
    assert q == num / (float(two_m) * float(two_m))
