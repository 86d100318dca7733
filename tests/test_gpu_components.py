"""APSP(C) of components between 256 vertices (one workgroup each) and a few
thousand (multi-workgroup rounds): those of one padded size are closed as a
batch wherever they lie among the others.  Every table equals the one-by-one
closure's (plain) and, on some, a plain Floyd-Warshall."""
import numpy as np
import pytest

from paper_1503_07192_amd import spq

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


@pytest.mark.parametrize("sizes", [
    [257],
    [256, 257, 1, 384, 385, 256, 385, 64],
    [512, 30, 513, 512, 640, 641, 512],
    [1024, 1025, 900, 1024, 5, 1023],
    [300] * 70,                       # many of one size
    [1100, 700, 1100, 700, 1100],     # sizes that alternate
])
def test_component_tables(sizes):
    rng = np.random.default_rng(len(sizes) + sizes[0])
    n, k = sum(sizes), len(sizes)
    part = np.repeat(np.arange(k), sizes)
    first = np.concatenate([[0], np.cumsum(sizes)])
    eu, ev = [], []
    for c, s in enumerate(sizes):
        if s == 1:
            continue
        a = rng.permutation(s) + first[c]              # a long path, then chords
        eu += [a[:-1], rng.integers(0, s, s) + first[c]]
        ev += [a[1:], rng.integers(0, s, s) + first[c]]
    eu += [first[:-2]] if k > 1 else []                # and edges between components
    ev += [first[1:-1] + np.array(sizes[1:]) // 2] if k > 1 else []
    eu, ev = np.concatenate(eu), np.concatenate(ev)
    w = rng.integers(0, 1000, len(eu))
    ids = rng.permutation(n)                           # vertex ids in no order
    eu, ev, p2 = ids[eu], ids[ev], np.empty(n, int)
    p2[ids] = part
    print("sizes", sizes[:8], flush=True)
    args = (n, dev(eu), dev(ev), dev(w), dev(p2), k)
    idx, one = spq.build_index(*args), spq.build_index(*args, plain=True)
    lo = spq.index_layout(idx)["local"]
    for c, s in enumerate(sizes):
        got = spq.index_component(idx, c, s)
        assert np.array_equal(got, spq.index_component(one, c, s)), c
        if c < 2 and s <= 700:
            d = np.full((s, s), spq.SPQ_INF, np.int64)
            np.fill_diagonal(d, 0)
            i = (p2[eu] == c) & (p2[ev] == c)
            np.minimum.at(d, (lo[eu[i]], lo[ev[i]]), w[i])
            np.minimum.at(d, (lo[ev[i]], lo[eu[i]]), w[i])
            np.fill_diagonal(d, 0)
            for x in range(s):
                d = np.minimum(d, d[:, x:x + 1] + d[x:x + 1])
            assert np.array_equal(got, np.minimum(d, spq.SPQ_INF)), c
