"""The path walk at the edges of its steps: vertices with more neighbours than
one group of eight, components whose boundary is wider than the minima kept in
LDS (1,024), no boundary at all, a walk across many components of one group and
of several, and a share.  Every path is checked against Dijkstra distances.
"""
import numpy as np
import pytest

from paper_1503_07192_amd import workloads as W

torch = pytest.importorskip("torch")
spq = pytest.importorskip("paper_1503_07192_amd.spq")

from test_gpu_parity import build  # noqa: E402
from test_gpu_paths import check_paths  # noqa: E402

pytestmark = pytest.mark.gpu


def graph(n, eu, ev, w, part, k, name):
    return dict(name=name, n=n, eu=np.asarray(eu, np.int32), ev=np.asarray(ev, np.int32),
                w=np.asarray(w, np.int32), part=np.asarray(part, np.int32), k=k)


def hubs(deg, wlo):
    """Two hubs over deg leaves each, the leaves joined in a cycle across components."""
    n = 2 + 2 * deg
    rng = np.random.default_rng(deg)
    leaves = np.arange(2, n)
    eu = np.concatenate([np.repeat([0, 1], deg), leaves])
    ev = np.concatenate([leaves, np.roll(leaves, 1)])
    return graph(n, eu, ev, rng.integers(wlo, 4, len(eu)), rng.integers(0, 5, n), 5, f"hub{deg}")


def strip(cols, rows, k, wlo=1):
    rng = np.random.default_rng(cols)
    eu, ev, w = W.random_grid(rng, cols, rows, keep=0.95, diag=0.3, wlo=wlo, whi=9)
    n = cols * rows
    return graph(n, eu, ev, w, np.arange(n) * k // n, k, f"strip{cols}x{rows}")


def interleaved(n):
    """A cycle with chords whose vertices alternate between two components: all on the boundary."""
    i = np.arange(n)
    rng = np.random.default_rng(n)
    eu, ev = np.concatenate([i, i]), np.concatenate([(i + 1) % n, rng.permutation(n)])
    return graph(n, eu, ev, rng.integers(1, 1000, 2 * n), i % 2, 2, f"alternating{n}")


CASES = [(hubs(7, 1), {}), (hubs(8, 1), {}), (hubs(9, 0), {}), (hubs(300, 0), {}),
         (strip(40, 30, 1), {}), (strip(33, 31, 25), dict(bg_method=2, group_comps=2)),
         (strip(31, 33, 9, 0), dict(bg_method=2, group_comps=9)),
         (strip(36, 20, 12), dict(share_comps=6, group_comps=3)),
         (interleaved(2046), {}), (interleaved(2050), {})]


@pytest.mark.parametrize("g,opts", CASES, ids=[c[0]["name"] for c in CASES])
def test_walk_steps(g, opts):
    idx = build(g, paths=True, **opts)
    rng = np.random.default_rng(3)
    own = np.flatnonzero(g["part"] < opts.get("share_comps", g["k"]))
    v1 = rng.choice(own, 600).astype(np.int32)
    v2 = rng.integers(0, g["n"], 600).astype(np.int32)
    # 300 leaves at distance 0 of a hub are more dead ends than a walk remembers
    # (16): such a walk may report -3, the others may not
    stall = g["name"] == "hub300"
    lens, stalled = check_paths(g, idx, v1, v2, 2 * g["n"], allow_stall=stall)
    assert stall or stalled == 0
    again, _ = check_paths(g, idx, v1, v2, 2 * g["n"], allow_stall=stall)
    assert (again == lens).all()
