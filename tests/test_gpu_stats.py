"""spq_index_stats reads what the build or replay left in host memory: it waits
for its own index only and queues nothing on the device."""
import numpy as np
import pytest

from paper_1503_07192_amd import spq, workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


def case(seed, side=64):
    rng = np.random.default_rng(seed)
    eu, ev, w = W.random_grid(rng, side, side, keep=0.97, diag=0.5, wlo=0, whi=1000)
    part, k = W.block_partition(side, side, 8, 8, 1)
    return side * side, eu, ev, w, part, k


def grid32():
    g = W.grid32()
    return g["eu"], g["ev"], g["w"], g["part"]


TWO_LEVEL = dict(bg_method=2, group_comps=8)


@pytest.mark.parametrize("opts", [dict(bg_method=1), TWO_LEVEL, dict(TWO_LEVEL, share_comps=16),
                                  dict(TWO_LEVEL, level3_groups=2)])
def test_stats_do_not_wait_for_other_work(opts):
    import torch
    n, eu, ev, w, part, k = case(1)
    ix = spq.build_index(n, dev(eu), dev(ev), dev(w), dev(part), k, **opts)
    first = spq.index_stats(ix)
    x = torch.zeros(1 << 28, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for _ in range(400):  # 2 GiB each way: more than 0.1 s in all
        x.add_(1)
    behind = torch.cuda.Event()
    behind.record()
    second = spq.index_stats(ix)
    assert not behind.query()
    torch.cuda.synchronize()
    assert first == second and first["relax_bg_exec"] > 0


def test_counts_of_replays_are_their_own():
    """Captured: every replay's products are counted anew (the same weights again
    give the first counts again; how many squarings a closure takes may differ by
    one or two, as they run in place)."""
    n, eu, ev, w, part, k = case(2)
    ix = spq.build_index(n, dev(eu), dev(ev), dev(w), dev(part), k, graph=True, level3_groups=2, **TWO_LEVEL)
    first = spq.index_stats(ix)
    rng = np.random.default_rng(3)
    for _ in range(3):
        spq.reweight(ix, dev(rng.integers(1, 1 << 20, len(w))))
        spq.index_stats(ix)
        spq.reweight(ix, dev(w))
        again = spq.index_stats(ix)
        assert again["relax_dominant"] == first["relax_dominant"] > 0
        assert abs(again["relax_bg_exec"] / first["relax_bg_exec"] - 1) < 0.5
        assert again["relax_comp_exec"] == first["relax_comp_exec"]


def squarings(executed, rows, used):
    """How many squarings of a block of `rows` rows, `used` of them vertices, make
    so many relaxations: whole 32-tiles of the upper triangle, each over all rows."""
    t = -(-used // 32)
    each = t * (t + 1) // 2 * 1024 * rows
    assert executed % each == 0, (executed, each)
    return executed // each


def test_squarings_that_end_at_once_are_not_counted():
    """A whole matrix of up to 512 vertices is closed by squarings, 9 of them planned;
    the ones after the first that lowers nothing do no work.  Edges between all pairs
    of weights in [500, 1000): no two of them are shorter than a third, and the first
    squaring finds nothing."""
    rng = np.random.default_rng(4)
    # two components of 400 vertices, closed in a batch of two, joined by 40 edges
    u, v = np.triu_indices(400, 1)
    eu = np.concatenate([u, u + 400, np.arange(40)])
    ev = np.concatenate([v, v + 400, np.arange(40) + 400])
    w = rng.integers(500, 1000, len(eu))
    part = np.arange(800) // 400
    ix = spq.build_index(800, dev(eu), dev(ev), dev(w), dev(part), 2, bg_method=1)
    st = spq.index_stats(ix)
    assert st["v_bg"] == 80
    assert squarings(int(st["relax_comp_exec"]), 512, 512) == 2  # one of each
    flat = spq.build_index(1024, *[dev(x) for x in grid32()], 16, bg_method=1)
    st = spq.index_stats(flat)
    assert st["v_bg_padded"] == 384
    assert squarings(int(st["relax_bg_exec"]), 384, 384) in range(2, 9)
