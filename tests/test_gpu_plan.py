"""The automatic plan (method, components per group, level 3): whatever it picks,
the index answers as the flat closure's does, row for row and pair for pair,
over the forms of partition it decides on: compact and strip-shaped groups,
partitions that cut everywhere, one component far larger than the rest, many
components without any boundary, odd and ragged sizes; captured builds and their
replays, certified weights and the path walk included."""
import numpy as np
import pytest

from paper_1503_07192_amd import spq, workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


def grid(seed, rows, cols, br, bc, order=1, wmax=1000):
    rng = np.random.default_rng(seed)
    eu, ev, w = W.random_grid(rng, rows, cols, keep=0.97, diag=0.5, wlo=0, whi=wmax)
    part, k = W.block_partition(rows, cols, br, bc, order)
    return rows * cols, eu, ev, w, part, k


def shuffled(g):
    n, eu, ev, w, part, k = g
    return n, eu, ev, w, np.random.default_rng(3).permutation(part), k


def one_large(g):
    """Components 0 .. k/2 - 1 merged into one, the others renumbered after it."""
    n, eu, ev, w, part, k = g
    return n, eu, ev, w, np.maximum(part - (k // 2 - 1), 0).astype(np.int32), k - k // 2 + 1


def isolated(g, extra):
    """`extra` more vertices, each a component of its own without any edge,
    between the first component and the others."""
    n, eu, ev, w, part, k = g
    part = np.where(part > 0, part + extra, 0)
    return n + extra, eu, ev, w, np.concatenate([part, 1 + np.arange(extra)]).astype(np.int32), k + extra


CASES = {
    # name: graph, method expected (None: either)
    "rows": (grid(1, 64, 64, 8, 8), 2),
    "z_order": (grid(2, 80, 80, 8, 8, 0), 2),
    "ragged": (grid(3, 91, 67, 7, 5), None),
    "strips": (grid(4, 40, 200, 40, 5), None),
    "shuffled": (shuffled(grid(5, 48, 48, 8, 8)), 1),
    "one_large": (one_large(grid(6, 64, 96, 8, 8)), None),
    "isolated": (isolated(grid(7, 64, 64, 8, 8), 700), None),
    "tiny_components": (grid(8, 48, 40, 1, 2), None),
    "small": (grid(9, 24, 24, 8, 8), 1),
    "level3": (grid(10, 130, 130, 8, 8), 2),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_planned_index_equals_flat(name):
    (n, eu, ev, w, part, k), method = CASES[name]
    a = [dev(x) for x in (eu, ev, w, part)]
    print("case", name, "n", n, "k", k, flush=True)
    flat = spq.build_index(n, *a, k, bg_method=1)
    auto = spq.build_index(n, *a, k)
    st = spq.index_stats(auto)
    print({x: st[x] for x in ("v_bg", "bg_method", "ngroups", "v_bg2", "groups3")}, flush=True)
    assert method is None or st["bg_method"] == method
    V = st["v_bg"]
    for r in np.random.default_rng(1).integers(0, V, 25):
        assert np.array_equal(spq.index_bg_rows(auto, int(r), 1, V), spq.index_bg_rows(flat, int(r), 1, V))
    rng = np.random.default_rng(2)
    v1, v2 = dev(rng.integers(0, n, 30000)), dev(rng.integers(0, n, 30000))
    want = spq.query_batch(flat, v1, v2)
    assert bool((spq.query_batch(auto, v1, v2) == want).all())


@pytest.mark.parametrize("side,method", [(72, 1), (96, 2)])
@pytest.mark.parametrize("wmax", [1000, 10_000_000])
def test_planned_captured_build_and_replay(wmax, side, method):
    """wmax 1e7: the total weight is past int32, the build certifies itself."""
    n, eu, ev, w, part, k = grid(11, side, side, 8, 8, wmax=wmax)
    rng = np.random.default_rng(4)
    v1, v2 = dev(rng.integers(0, n, 20000)), dev(rng.integers(0, n, 20000))
    a = [dev(eu), dev(ev), dev(w), dev(part)]
    auto = spq.build_index(n, *a, k, graph=True, paths=True)
    assert spq.index_stats(auto)["bg_method"] == method
    for i in range(3):
        w2 = dev(rng.permutation(w))
        spq.reweight(auto, w2)
        flat = spq.build_index(n, a[0], a[1], w2, a[3], k, bg_method=1)
        assert bool((spq.query_batch(auto, v1, v2) == spq.query_batch(flat, v1, v2)).all()), i
        flat.free()
    paths, lens = spq.query_paths(auto, v1[:200], v2[:200], n)
    assert int(lens.min()) >= 0
