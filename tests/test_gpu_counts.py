"""The counters per component (sizes, boundary sizes, weights inside, slots of
the renumbering), raised for a wave's lanes of one component at once: the layout
must be the plain one (boundary first, ascending ids) for runs of every length
around the grouping's limits (four lanes, four components per wave), components
that alternate, one component, sizes around a wave, and the component matrices
must start from the lightest edge (all-pairs of tiny components)."""
import numpy as np
import pytest

from paper_1503_07192_amd import spq

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


def runs(n, length, k):
    return (np.arange(n) // length) % k


PARTS = {
    "one": lambda n, rng: np.zeros(n, int),
    "runs3": lambda n, rng: runs(n, 3, max(1, n // 40)),
    "runs4": lambda n, rng: runs(n, 4, max(1, n // 40)),
    "runs5": lambda n, rng: runs(n, 5, max(1, n // 40)),
    "runs13": lambda n, rng: runs(n, 13, max(1, n // 40)),
    "alternate": lambda n, rng: np.arange(n) % 2 if n > 1 else np.zeros(n, int),
    "random": lambda n, rng: rng.permutation(np.arange(n) % max(1, n // 20)),
    "skewed": lambda n, rng: np.where(rng.random(n) < 0.9, 0, 1 + np.arange(n) % max(1, n // 20)),
}


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257, 3000])
@pytest.mark.parametrize("name", sorted(PARTS))
def test_layout_is_plain(name, n):
    rng = np.random.default_rng(n)
    part = PARTS[name](n, rng)
    _, part = np.unique(part, return_inverse=True)
    k = int(part.max()) + 1
    m = 3 * n
    eu, ev = rng.integers(0, n, m), rng.integers(0, n, m)
    near = rng.random(m) < 0.6           # most edges inside a component
    order = np.argsort(part, kind="stable")
    place = np.empty(n, int)
    place[order] = np.arange(n)
    ev = np.where(near, order[np.minimum(place[eu] + 1, n - 1)], ev)
    w = rng.integers(0, 1000, m)
    print("case", name, n, "k", k, flush=True)
    idx = spq.build_index(n, dev(eu), dev(ev), dev(w), dev(part), k)
    lay = spq.index_layout(idx)
    cross = part[eu] != part[ev]
    b = np.zeros(n, bool)
    b[eu[cross]] = True
    b[ev[cross]] = True
    nb = np.bincount(part[b], minlength=k)
    size = np.bincount(part, minlength=k)
    assert np.array_equal(lay["comp"], part)
    assert np.array_equal(lay["nb"], nb)
    assert np.array_equal(lay["off"], np.concatenate([[0], np.cumsum(size)]))
    assert np.array_equal(lay["bgoff"], np.concatenate([[0], np.cumsum(nb)]))
    for c in range(k):
        ids = np.flatnonzero(part == c)
        want = np.concatenate([ids[b[ids]], ids[~b[ids]]])
        got = np.empty(len(ids), int)
        got[lay["local"][ids]] = ids
        assert np.array_equal(got, want), c
    # one component's closure against a plain Floyd-Warshall
    c = int(np.argmax(np.where(size <= 300, size, 0)))
    if size[c] <= 300:
        ids = np.flatnonzero(part == c)
        d = np.full((len(ids), len(ids)), spq.SPQ_INF, np.int64)
        np.fill_diagonal(d, 0)
        ins = (part[eu] == c) & (part[ev] == c)
        lo = lay["local"]
        np.minimum.at(d, (lo[eu[ins]], lo[ev[ins]]), w[ins])
        np.minimum.at(d, (lo[ev[ins]], lo[eu[ins]]), w[ins])
        for x in range(len(ids)):
            d = np.minimum(d, d[:, x:x + 1] + d[x:x + 1])
        assert np.array_equal(spq.index_component(idx, c, len(ids)), np.minimum(d, spq.SPQ_INF))
    idx.free()


def test_component_weight_past_int32_is_refused():
    """Weights inside one component summing past int32, spread over a wave and
    over several: counted exactly (the build refuses such a component)."""
    n = 200
    eu, ev = np.arange(n - 1), np.arange(1, n)
    for w, ok in ((2**31 // n, True), (2**31 // (n - 1) + 1, False)):
        args = (n, dev(eu), dev(ev), dev(np.full(n - 1, w)), dev(np.zeros(n)), 1)
        if ok:
            spq.build_index(*args).free()
        else:
            with pytest.raises(spq.SpqError) as e:
                spq.build_index(*args)
            assert e.value.name == "SPQ_ERANGE"
