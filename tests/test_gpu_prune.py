"""The composition's pruning on operands that it does prune: distances between
points of a plane (a group's boundary reached from far away), against the
oracle's plain (min, +) product, bit-exact.

The sizes sit at the edges of the kernels: boundary counts around a mask word
(64), a list window (256), an LDS segment of the masks (4,096) and the statistics' sample
(16 rows); vertex counts around the row and column tiles (64, 128); rows that
are INF on the sampled boundary rows only, and rows and columns that nothing
reaches.
"""
import numpy as np
import pytest

import oracle
from oracle import O_INF
from paper_1503_07192_amd import spq

pytestmark = pytest.mark.gpu
INF = spq.SPQ_INF


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


def to64(a):
    a = np.asarray(a, np.int64)
    return np.where(a >= INF, O_INF, a)


def plane_case(seed, nv, nk, scale):
    """Groups of points in unit squares 3 apart; distances scaled to integers."""
    rng = np.random.default_rng(seed)
    G = len(nv)
    vp = -(-max(nv) // 128) * 128
    kp = -(-max(max(nk), 1) // 128) * 128
    pts = [rng.random((v, 2)) + [3.0 * g, 0] for g, v in enumerate(nv)]
    bnd = [rng.random((k, 2)) + [3.0 * g, 0] for g, k in enumerate(nk)]
    dist = lambda p, q: np.rint(np.hypot(*(p[:, None] - q[None]).transpose(2, 0, 1)) * scale).astype(np.int64)
    allb = np.concatenate(bnd)
    D = dist(allb, allb)
    R = rng.integers(0, INF, (G, kp, vp), dtype=np.int64)
    M = rng.integers(0, INF, (G, vp, vp), dtype=np.int64)
    for g in range(G):
        R[g, :nk[g], :nv[g]] = dist(bnd[g], pts[g])
        M[g, :nv[g], :nv[g]] = dist(pts[g], pts[g])
    return vp, kp, R, D, M


def check(nv, nk, vp, kp, R, D, M, layout):
    import torch
    G = len(nv)
    koff = np.concatenate([[0], np.cumsum(nk)])
    voff = np.concatenate([[0], np.cumsum(nv)])
    pairs = [(a, b) for a in range(G) for b in range(a, G)]
    nv, nk = np.array(nv, np.int32), np.array(nk, np.int32)
    ldd = D.shape[1]
    if layout == spq.SPQ_MP_DENSE:
        out = torch.full((int(voff[-1]), int(voff[-1])), -7, dtype=torch.int32, device="cuda")
        spq.minplus_batched(layout, nv, nk, vp, kp, dev(R), dev(D), ldd, dev(M), pairs, out,
                            ldo=int(voff[-1]))
    else:
        out = torch.full((sum(int(nv[a]) * int(nv[b]) for a, b in pairs),), -7, dtype=torch.int32,
                         device="cuda")
        spq.minplus_batched(layout, nv, nk, vp, kp, dev(R), dev(D), ldd, dev(M), pairs, out,
                            cb=int(nv.max()))
    got = out.cpu().numpy()
    base = 0
    for a, b in pairs:
        Db = to64(D[koff[a]:koff[a + 1], koff[b]:koff[b + 1]])
        T = oracle.minplus(oracle.minplus(to64(R[a, :nk[a], :nv[a]]).T.copy(), Db),
                           to64(R[b, :nk[b], :nv[b]]))
        if a == b:
            T = np.minimum(T, to64(M[a, :nv[a], :nv[a]]))
        T = np.minimum(T, INF)
        if layout == spq.SPQ_MP_DENSE:
            block = got[voff[a]:voff[a + 1], voff[b]:voff[b + 1]]
        else:  # one run per group: the block is row-major
            n = int(nv[a]) * int(nv[b])
            block = got[base:base + n].reshape(nv[a], nv[b])
            base += n
        assert np.array_equal(block, T), (a, b)


@pytest.mark.parametrize("layout", [spq.SPQ_MP_BLOCKED, spq.SPQ_MP_DENSE])
@pytest.mark.parametrize("nv,nk", [
    ([64, 65, 1], [63, 64, 65]),
    ([127, 128, 129], [15, 16, 17]),
    ([200, 63], [255, 257]),
    ([130, 70], [256, 512]),
    ([40, 30], [4097, 4096]),
])
def test_plane_products_equal_oracle(nv, nk, layout):
    vp, kp, R, D, M = plane_case(sum(nv) + sum(nk), nv, nk, 1e5)
    print("case", nv, nk, layout, flush=True)
    check(nv, nk, vp, kp, R, D, M, layout)


@pytest.mark.parametrize("scale", [1.0, 3e8, 2e9])
def test_plane_products_at_the_ends_of_the_range(scale):
    """Ties everywhere (distances 0 .. 6), and distances up to and past INF."""
    nv, nk = [100, 90, 70], [80, 40, 130]
    vp, kp, R, D, M = plane_case(7, nv, nk, scale)
    R, D, M = (np.minimum(x, INF) for x in (R, D, M))
    print("scale", scale, flush=True)
    check(nv, nk, vp, kp, R, D, M, spq.SPQ_MP_BLOCKED)


def test_unreachable_rows_and_columns():
    """Rows INF on every k, on the sampled k only and on all but one k; columns
    likewise."""
    nv, nk = [100, 130], [70, 90]
    vp, kp, R, D, M = plane_case(11, nv, nk, 1e5)
    ko = nk[0]
    R[0, :nk[0], 5] = INF            # a vertex no boundary vertex reaches
    R[1, :nk[1], 64:129] = INF       # a column tile of them
    sampled = [i * nk[0] // 16 for i in range(16)]
    D[sampled, ko + 3] = INF         # a row of the first product: INF where it is sampled
    D[:ko, ko + 7] = INF
    D[:ko, ko + 9] = INF
    D[33, ko + 9] = 5
    R[1, :nk[1], 2] = INF
    R[1, 8, 2] = 1
    for layout in (spq.SPQ_MP_BLOCKED, spq.SPQ_MP_DENSE):
        print("layout", layout, flush=True)
        check(nv, nk, vp, kp, R, D, M, layout)
