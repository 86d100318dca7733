"""The dense closure's pivot blocks, closed by squarings, and its launches split
into 64-tiles, on the inputs with the longest shortest paths: one path through
all vertices, its vertices shuffled, so that the shortest walk between its ends
has v - 1 steps (closed form: differences of prefix sums), and the same with a
second component.  Sizes around the squared blocks (32-row tiles, 256 and 512
rows, whole matrices up to 512) and the rounds beyond."""
import numpy as np
import pytest

from paper_1503_07192_amd import spq

pytestmark = pytest.mark.gpu
INF = spq.SPQ_INF


@pytest.mark.parametrize("tile,pivot", [(128, 1), (128, 2), (128, 4), (64, 2), (64, 4)])
@pytest.mark.parametrize("v", [2, 33, 129, 256, 257, 384, 511, 512, 513, 900])
def test_shuffled_path_closure(tile, pivot, v):
    import torch
    rng = np.random.default_rng(v * 8 + pivot)
    ld = -(-v // tile) * tile
    order = rng.permutation(v)
    w = rng.integers(0, 1000, v - 1).astype(np.int64)
    cut = rng.integers(0, v - 1) if v > 300 else -1   # the edge left out, if any
    m = np.full((ld, ld), INF, np.int64)
    np.fill_diagonal(m, 0)
    for i in range(v - 1):
        if i != cut:
            a, b = order[i], order[i + 1]
            m[a, b] = m[b, a] = w[i]
    pre = np.concatenate([[0], np.cumsum(w)])
    side = np.arange(v) > cut if cut >= 0 else np.zeros(v, bool)
    want = np.full((ld, ld), INF, np.int64)
    np.fill_diagonal(want, 0)
    d = np.abs(pre[:, None] - pre[None, :])
    d[side[:, None] != side[None, :]] = INF
    want[np.ix_(order, order)] = d
    print("tile", tile, "pivot", pivot, "v", v, flush=True)
    t = torch.from_numpy(m.astype(np.int32)).cuda()
    spq.fw_dense(v, ld, tile, t, pivot=pivot * tile)
    assert np.array_equal(t.cpu().numpy(), want)
