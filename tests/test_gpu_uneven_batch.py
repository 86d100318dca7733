"""Batches of closures whose matrices differ in size: groups of 1,600 vertices beside
groups of 100, 37 and 1 in the same padded matrices, as groups, as super-groups and as
a share's blocks, on either side of each pivot rows option.
"""
import numpy as np
import pytest

import oracle
from paper_1503_07192_amd import workloads as W

torch = pytest.importorskip("torch")
spq = pytest.importorskip("paper_1503_07192_amd.spq")

from test_gpu_parity import INF32, build, dev  # noqa: E402

pytestmark = pytest.mark.gpu


def uneven(singles, first):
    """A 50-row grid: 50 columns in 100 blocks of 5 x 5, `singles` vertices one
    component each (first: they lead the component order), the rest one component."""
    cols = 50 + (singles + 49) // 50 + 4
    rng = np.random.default_rng(singles)
    eu, ev, w = W.random_grid(rng, cols, 50, keep=0.97, diag=0.2, wlo=1, whi=1000)
    n = cols * 50
    v = np.arange(n)
    if np.any(np.maximum(eu, ev) >= n):
        raise ValueError("grid order")
    x, y = v % cols, v // cols
    part = np.full(n, -1)
    left = x < 50
    part[left] = (y[left] // 5) * 10 + x[left] // 5
    rest = np.flatnonzero(~left)
    part[rest[:singles]] = 100 + np.arange(singles)
    part[rest[singles:]] = 100 + singles
    k = 101 + singles
    if first:
        part = (part + singles) % k
    return dict(name=f"uneven{singles}", n=n, eu=eu, ev=ev, w=w, part=part.astype(np.int32), k=k)


@pytest.mark.parametrize("singles,first,opts", [
    (737, False, dict(group_comps=100)), (737, True, dict(group_comps=100)),
    (500, False, dict(group_comps=100, level3_groups=2)), (537, True, dict(group_comps=50, level3_groups=3)),
    (300, False, dict(group_comps=50, share_comps=50)), (300, True, dict(group_comps=100, share_comps=300))])
def test_uneven_batches(singles, first, opts):
    g = uneven(singles, first)
    idx = build(g, bg_method=2, **opts)
    rng = np.random.default_rng(1)
    own = np.flatnonzero(g["part"] < opts.get("share_comps", g["k"]))
    src = rng.choice(own, 60, replace=False).astype(np.int32)
    v1, v2 = np.repeat(src, g["n"]).astype(np.int32), np.tile(np.arange(g["n"], dtype=np.int32), 60)
    got = spq.query_batch(idx, dev(v1), dev(v2)).cpu().numpy().reshape(60, -1)
    D = oracle.dijkstra(g["n"], g["eu"], g["ev"], g["w"], src)
    assert (got == np.minimum(D, INF32)).all()
