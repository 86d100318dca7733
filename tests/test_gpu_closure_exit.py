"""Block closures that end before their last squaring, and ones that need every
squaring: a path (hops across the whole block), a star (two hops), a closed
clique (none).  Reweighting replays the captured closures, so each replay starts
from the flags of the one before.
"""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
spq = pytest.importorskip("paper_1503_07192_amd.spq")

from test_gpu_parity import INF32, build, dev  # noqa: E402

pytestmark = pytest.mark.gpu


def shape(kind, n, rng):
    i = np.arange(n)
    if kind == "path":
        order = rng.permutation(n)
        return order[:-1], order[1:]
    if kind == "line":
        return i[:-1], i[1:]
    if kind == "star":
        return np.zeros(n - 1, int), i[1:]
    u, v = np.triu_indices(n, 1)
    return u, v


@pytest.mark.parametrize("kind,n", [("path", 129), ("line", 256), ("path", 400), ("line", 512), ("star", 257),
                                    ("clique", 300), ("path", 513), ("line", 1100), ("star", 1100),
                                    ("clique", 700)])
def test_closure_exit(kind, n):
    rng = np.random.default_rng(n)
    eu, ev = (np.asarray(x, np.int32) for x in shape(kind, n, rng))
    w = rng.integers(1000, 2000, len(eu)).astype(np.int32)  # a clique of these is closed
    g = dict(name=kind, n=n, eu=eu, ev=ev, w=w, part=np.arange(n, dtype=np.int32), k=n)
    idx = build(g, graph=True, bg_method=1)
    src = rng.integers(0, n, 40).astype(np.int32)
    v1, v2 = np.repeat(src, n).astype(np.int32), np.tile(np.arange(n, dtype=np.int32), 40)
    for step in range(5):
        got = spq.query_batch(idx, dev(v1), dev(v2)).cpu().numpy()
        D = oracle.dijkstra(n, eu, ev, w, src)
        assert (got == np.minimum(D, INF32).reshape(-1)).all(), step
        lo = 1 if step % 2 == 0 else 1000  # every other time not closed before
        w = rng.integers(lo, 2000, len(eu)).astype(np.int32)
        spq.reweight(idx, dev(w))
