"""A share's last Bellman-Ford product over the k that can matter: few and many share
sources (one tile, a remainder, several), blocks without rows outside their boundary,
blocks nothing enters, zero weights and ties.  Against Dijkstra.
"""
import numpy as np
import pytest

import oracle
from paper_1503_07192_amd import workloads as W

torch = pytest.importorskip("torch")
spq = pytest.importorskip("paper_1503_07192_amd.spq")

from test_gpu_parity import INF32, build, dev  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,br,share,group,blk,wlo,whi,cut", [
    (32, 32, 4, 1, 1, 4, 1, 100, False), (48, 40, 4, 8, 2, 4, 1, 1, False), (64, 64, 4, 40, 4, 4, 0, 3, False),
    (64, 64, 8, 16, 1, 1, 1, 1000, False), (96, 64, 4, 100, 6, 2, 1, 10**5, False),
    (64, 48, 4, 20, 3, 5, 0, 50, True), (40, 40, 4, 100, 10, 3, 1, 9, True)])
def test_share_rows(rows, cols, br, share, group, blk, wlo, whi, cut):
    rng = np.random.default_rng(rows * cols + share)
    eu, ev, w = W.random_grid(rng, rows, cols, keep=0.96, diag=0.2, wlo=wlo, whi=whi)
    if cut:  # two halves without an edge between them
        keep = (eu // cols < rows // 2) == (ev // cols < rows // 2)
        eu, ev, w = eu[keep], ev[keep], w[keep]
    part, k = W.block_partition(rows, cols, br, br)
    g = dict(name="rows", n=rows * cols, eu=eu, ev=ev, w=w, part=part, k=k)
    idx = build(g, bg_method=2, group_comps=group, share_comps=share, level3_groups=blk)
    own = np.flatnonzero(np.asarray(part) < share)
    src = rng.choice(own, min(50, len(own)), replace=False).astype(np.int32)
    v1, v2 = np.repeat(src, g["n"]).astype(np.int32), np.tile(np.arange(g["n"], dtype=np.int32), len(src))
    got = spq.query_batch(idx, dev(v1), dev(v2)).cpu().numpy().reshape(len(src), -1)
    assert (got == np.minimum(oracle.dijkstra(g["n"], eu, ev, w, src), INF32)).all()
