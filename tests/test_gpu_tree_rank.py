"""The tree layout above and below the size from which its walk is ranked by splitters (2^14 arcs), on the shapes
where the walk's next arc lies far from or right beside the current one, and on marks that are no spanning tree."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def tree_edges(kind, n, rng):
    """A tree on n nodes whose ids are shuffled (except the path's)."""
    i = np.arange(1, n)
    par = {"path": i - 1, "star": np.zeros(n - 1, int), "random": rng.integers(0, i), "binary": (i - 1) // 2,
           "caterpillar": np.where(i % 2 == 1, np.maximum(i - 2, 0), i - 1)}[kind]
    ids = np.arange(n) if kind == "path" else rng.permutation(n)
    a, b = ids[i], ids[par]
    key = np.sort(np.minimum(a, b).astype(np.int64) * n + np.maximum(a, b))
    return (key // n).astype(np.int32), (key % n).astype(np.int32), rng.uniform(0.5, 2.0, n - 1)


# 8192 nodes: 16382 arcs, just below the bound; 8193: 16384; ragged last buckets on both levels
@pytest.mark.parametrize("n", [8192, 8193, 8200, 50021, 300007])
@pytest.mark.parametrize("kind", ["path", "star", "random", "binary", "caterpillar"])
def test_walk_order(orc, kind, n):
    from paper_2008_07633_amd import sfg as S

    u, v, w = tree_edges(kind, n, np.random.default_rng(660 + n))
    t = S.sfg_tree_order(n, dev(u), dev(v), dev(w), torch.ones(n - 1, dtype=torch.uint8, device="cuda"))
    want = orc.tree_dfs(n, u, v, w, np.ones(n - 1, bool))
    for name in ("order", "parent", "size", "tdown", "tup", "pw"):
        assert np.array_equal(getattr(t, name).cpu().numpy(), getattr(want, name)), name


@pytest.mark.parametrize("n", [9000, 60000])
@pytest.mark.parametrize("ring", [3, 64, 2000])
def test_marks_with_a_ring(n, ring):
    # a ring apart from a path through the root: n - 1 marked edges, two components
    from paper_2008_07633_amd import sfg as S

    m = n - ring
    u = np.r_[np.arange(m - 1), np.arange(m, n - 1), [m]]
    v = np.r_[np.arange(1, m), np.arange(m + 1, n), [n - 1]]
    o = np.lexsort((v, u))
    u, v = u[o].astype(np.int32), v[o].astype(np.int32)
    assert u.size == n - 1
    with pytest.raises(S.SfgError) as e:
        S.sfg_tree_order(n, dev(u), dev(v), dev(np.ones(n - 1)), torch.ones(n - 1, dtype=torch.uint8, device="cuda"))
    assert e.value.name == "SFG_ENOTCONN"


# 196608 nodes: 393214 arcs, the longest walk that is ranked by pointer jumping; splitters from 393216 on
@pytest.mark.parametrize("n", [196608, 196609, 200003])
@pytest.mark.parametrize("kind", ["path", "star", "random", "caterpillar"])
def test_walk_order_at_the_bound(orc, kind, n):
    test_walk_order(orc, kind, n)


@pytest.mark.parametrize("ring", [3, 64, 100000])
def test_marks_with_a_ring_by_splitters(ring):
    test_marks_with_a_ring(250000, ring)
