"""The composition's scratch: a built index does not keep it, and the next
build may have it while the first one's queued work still runs."""
import numpy as np
import pytest

from paper_1503_07192_amd import spq, workloads as W

pytestmark = pytest.mark.gpu
GIB = 1 << 30


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


def case(seed, side=256):
    rng = np.random.default_rng(seed)
    eu, ev, w = W.random_grid(rng, side, side, keep=0.97, diag=0.5, wlo=0, whi=1000)
    part, k = W.block_partition(side, side, 8, 8, 1)
    n = side * side
    return n, [dev(x) for x in (eu, ev, w, part)], k, dev(rng.integers(0, n, 20000)), dev(rng.integers(0, n, 20000))


@pytest.mark.parametrize("graph", [False, True])
def test_resident_indexes_hold_no_large_scratch(graph):
    """256 groups, 32,896 pairs: launches of up to 2 GiB of scratch beside a store
    of 1.4 GiB and BG2 of 1.2.  A second resident index takes these two, its other
    tables (below 0.5 GiB) and, captured, scratch for its replays of at most half
    of the two levels' output."""
    import torch
    n, a, k, v1, v2 = case(21)
    opts = dict(bg_method=2, group_comps=4, graph=graph)
    spq.release_cached_memory()
    first = spq.build_index(n, *a, k, **opts)
    want = spq.query_batch(first, v1, v2)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    second = spq.build_index(n, *a, k, **opts)
    got = spq.query_batch(second, v1, v2)
    torch.cuda.synchronize()
    taken = free - torch.cuda.mem_get_info()[0]
    st = spq.index_stats(second)
    print("graph", graph, "store", st["bg_bytes"], "taken", taken, st["ngroups"], st["groups3"], flush=True)
    bg2 = 4 * (st["v_bg2"] + 128) ** 2
    scratch = st["bg_bytes"] / 2 + bg2 / 4 if graph else 0
    assert taken < st["bg_bytes"] + bg2 + 0.5 * GIB + scratch
    assert bool((got == want).all())


def test_scratch_is_not_reused_while_work_on_it_is_queued():
    """Builds on two streams in turn, queries on each, no wait in between; then
    the cache is emptied behind them."""
    import torch
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    cases = [case(s, 192) for s in (31, 32)]
    want = []
    for n, a, k, v1, v2 in cases:
        flat = spq.build_index(n, *a, k, bg_method=1)
        want.append(spq.query_batch(flat, v1, v2))
        flat.free()
    torch.cuda.synchronize()
    held = []
    for rep in range(6):
        i = rep & 1
        n, a, k, v1, v2 = cases[i]
        with torch.cuda.stream(streams[i]):
            ix = spq.build_index(n, *a, k, bg_method=2, group_comps=4 << (rep % 3))
            held.append((i, ix, spq.query_batch(ix, v1, v2)))
    spq.release_cached_memory()
    torch.cuda.synchronize()
    for i, _, got in held:
        assert bool((got == want[i]).all())
