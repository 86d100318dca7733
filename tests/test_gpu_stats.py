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
    give the first counts again)."""
    n, eu, ev, w, part, k = case(2)
    ix = spq.build_index(n, dev(eu), dev(ev), dev(w), dev(part), k, graph=True, level3_groups=2, **TWO_LEVEL)
    keys = ("relax_comp_exec", "relax_bg_exec", "relax_dominant")
    first = spq.index_stats(ix)
    rng = np.random.default_rng(3)
    for _ in range(3):
        spq.reweight(ix, dev(rng.integers(1, 1 << 20, len(w))))
        spq.index_stats(ix)
        spq.reweight(ix, dev(w))
        again = spq.index_stats(ix)
        assert [again[x] for x in keys] == [first[x] for x in keys]
    assert first["relax_dominant"] > 0
