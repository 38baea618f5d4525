"""Spanning forests at the edges of the size rules: one-workgroup graphs (up to 8192 nodes and 32768 edges), lists
taken in one part and in two, ties on both sides of the split, long hook chains and disconnected graphs."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def random_list(n, m, rng):
    a, b = rng.integers(0, n, 2 * m + 64), rng.integers(0, n, 2 * m + 64)
    key = np.unique(np.minimum(a, b)[a != b] * n + np.maximum(a, b)[a != b])
    key = np.sort(rng.permutation(key)[:m])
    return (key // n).astype(np.int32), (key % n).astype(np.int32)


def check(orc, n, u, v, w, allowed=None):
    from paper_2008_07633_amd import sfg as S

    ref_t, ref_c = orc.max_spanning_forest(n, u, v, w, allowed=allowed)
    for dt in (torch.float64, torch.float32):
        if dt == torch.float32 and not np.array_equal(w.astype(np.float32).astype(np.float64), w):
            continue
        t, c = S.sfg_spanning_tree(n, dev(u), dev(v), dev(w).to(dt), allowed=None if allowed is None else dev(allowed))
        assert np.array_equal(t.cpu().numpy(), ref_t) and c == ref_c, dt


WEIGHTS = {
    "lognormal": lambda rng, m: rng.lognormal(0.0, 1.5, m).astype(np.float32).astype(np.float64),
    "unit": lambda rng, m: np.ones(m),
    "three": lambda rng, m: rng.integers(1, 4, m).astype(np.float64),
}


# around the one-workgroup limits; sparse (one part) and dense (two parts) lists; many components
@pytest.mark.parametrize("n,m", [(8192, 32768), (8193, 32768), (8192, 32769), (5, 4), (300, 8193), (50000, 60000),
                                 (20000, 400000), (60000, 90000), (200001, 700003)])
@pytest.mark.parametrize("weights", list(WEIGHTS))
def test_random_graphs(orc, n, m, weights):
    rng = np.random.default_rng(640 + n)
    u, v = random_list(n, m, rng)
    check(orc, n, u, v, WEIGHTS[weights](rng, u.size))


@pytest.mark.parametrize("n", [8000, 300000])
def test_monotone_path(orc, n):
    # every node hooks onto the next one: a single chain of n - 1 hooks in the first round
    for w in (np.arange(1.0, n), np.arange(float(n - 1), 0.0, -1.0)):
        check(orc, n, np.arange(n - 1, dtype=np.int32), np.arange(1, n, dtype=np.int32), w)


def test_star_with_chords(orc):
    # one component that almost every edge touches
    rng = np.random.default_rng(650)
    u, v = random_list(30000, 200000, rng)
    key = np.unique(np.r_[u.astype(np.int64) * 30000 + v, np.arange(1, 30000)])
    u, v = (key // 30000).astype(np.int32), (key % 30000).astype(np.int32)
    check(orc, 30000, u, v, rng.uniform(0.5, 2.0, u.size))


@pytest.mark.parametrize("share", [0.0, 0.02, 0.6])
def test_allowed_mask(orc, share):
    g = W.mesh3d(40, 37, 35, seed=651, wdist=("lognormal", 0.0, 1.5))
    allowed = (np.random.default_rng(652).random(g.m) < share).astype(np.uint8)
    check(orc, g.n, g.u, g.v, g.w, allowed)
