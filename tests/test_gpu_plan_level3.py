"""Which super-groups close BG2 (level 3) when the build chooses by itself."""
import numpy as np
import pytest

from paper_1503_07192_amd import spq, workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).cuda()


def build_and_check(side, **opts):
    """A side x side grid in 8 x 8 blocks; its index's statistics, answers
    compared with the flat closure's."""
    rng = np.random.default_rng(10)
    eu, ev, w = W.random_grid(rng, side, side, keep=0.97, diag=0.5, wlo=0, whi=1000)
    part, k = W.block_partition(side, side, 8, 8, 1)
    n = side * side
    a = [dev(x) for x in (eu, ev, w, part)]
    auto = spq.build_index(n, *a, k, **opts)
    st = spq.index_stats(auto)
    print(side, opts, {x: st[x] for x in ("v_bg", "ngroups", "v_bg2", "groups3", "v_bg3")}, flush=True)
    flat = spq.build_index(n, *a, k, bg_method=1)
    v1, v2 = dev(rng.integers(0, n, 30000)), dev(rng.integers(0, n, 30000))
    assert bool((spq.query_batch(auto, v1, v2) == spq.query_batch(flat, v1, v2)).all())
    return st


@pytest.mark.parametrize("side,groups,groups3", [(150, 46, 6), (230, 14, 7)])
def test_partial_last_group(side, groups, groups3):
    """361 components in groups of 8, 841 in groups of 64: the last group holds
    one and nine.  The cut of a super-group is counted for the components that a
    group holds (by the mean it came out as of half the width, and groups of 16
    and 4 were taken for 8 and 2)."""
    st = build_and_check(side)
    assert (st["ngroups"], st["groups3"]) == (groups, groups3)


@pytest.mark.parametrize("side,groups3", [(130, 0), (200, 5)])
def test_level3_is_taken_where_it_pays(side, groups3):
    """2,175 BG2 vertices: one flat closure is estimated at 1.2 ms, any
    super-groups at 1.6 or more.  7,643 of 20 groups: 11 ms flat, 3.1 by
    super-groups of 4."""
    st = build_and_check(side)
    assert st["groups3"] == groups3 and (st["v_bg3"] > 0) == (groups3 > 0)


@pytest.mark.parametrize("level3,groups,groups3", [(-1, 10, 0), (16, 79, 5), (0, 20, 5)])
def test_grouping_follows_the_callers_level3(level3, groups, groups3):
    """Groups are chosen for the closure of BG2 that the caller asks for: without
    level 3, half as many wider ones (3,600 BG2 vertices instead of 7,600), for
    super-groups of 16 four times as many."""
    st = build_and_check(200, level3_groups=level3)
    assert (st["ngroups"], st["groups3"]) == (groups, groups3)
