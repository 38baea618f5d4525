"""Sweeps and BF16 layers over the last rows of the largest graphs: entry indices up to 2^31 - 2, where a signed index
that steps over its row's end would wrap.  The graph's own rows stand for the last ones: their extents are moved to the
end of the index range and the arrays' addresses back by as much, so that every entry keeps its place in memory and
the results have to be those of the same rows at the start."""
import ctypes

import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def last_row(n, length):
    """A random graph whose last row has `length` entries, as (u, v, w)."""
    g = W.random_connected(n - 1, n, seed=900 + length)
    rng = np.random.default_rng(901 + length)
    hub = np.sort(rng.choice(n - 1, length, replace=False))
    key = np.sort(np.r_[g.u.astype(np.int64) * n + g.v, hub * n + (n - 1)])
    return (key // n).astype(np.int32), (key % n).astype(np.int32), rng.uniform(0.5, 2.0, key.size)


def at_the_end(G):
    """G with its entries at the end of the index range."""
    from paper_2008_07633_amd import sfg as S

    base = 2 ** 31 - 2 - G.nnz
    moved = (G.rowptr.long() + base).to(torch.int32)
    assert int(moved[-1]) == 2 ** 31 - 2

    class End(S.Csr):
        def struct(self):
            s = super().struct()
            s.rowptr = moved.data_ptr()
            s.col -= 4 * base
            s.eid -= 4 * base
            s.val -= self.val.element_size() * base
            return s

    return End(G.n, G.nnz, G.rowptr, G.col, G.val, G.eid, G.deg)


# the last row: taken by a lane group and, in reduced precision from 257 entries on, by a workgroup
@pytest.mark.parametrize("length", [3, 21, 257, 4096, 5000])
@pytest.mark.parametrize("dt,k", [(torch.float32, 16), (torch.float32, 12), (torch.float32, 5), (torch.float64, 16),
                                  (torch.bfloat16, 16), (torch.float16, 24)])
def test_sweeps(length, dt, k):
    from paper_2008_07633_amd import sfg as S

    n = 6000
    u, v, w = last_row(n, length)
    G = S.sfg_laplacian_csr(n, dev(u), dev(v), dev(w).to(torch.float64 if dt == torch.float64 else torch.float32))
    x0 = dev(np.random.default_rng(902).standard_normal((n, k)))
    want = S.sfg_smooth(G, x0, 3, storage=dt)
    assert torch.equal(S.sfg_smooth(at_the_end(G), x0, 3, storage=dt), want)
    if dt in (torch.float32, torch.float64):
        classes = S.sfg_color(G)
        want = S.sfg_smooth_gs(G, classes, x0, 2, storage=dt)
        assert torch.equal(S.sfg_smooth_gs(at_the_end(G), classes, x0, 2, storage=dt), want)


@pytest.mark.parametrize("per", [1, 6])
@pytest.mark.parametrize("length", [3, 21, 300])
def test_bf16_layers(length, per):
    from paper_2008_07633_amd import sfg as S

    n = 1000
    u, v, w = last_row(n, length)
    if per > 1:      # the dense form: more entries in flight
        g = W.random_connected(n - 1, per * n, seed=903)
        key = np.unique(np.r_[u.astype(np.int64) * n + v, g.u.astype(np.int64) * n + g.v])
        u, v = (key // n).astype(np.int32), (key % n).astype(np.int32)
        w = np.random.default_rng(904).uniform(0.5, 2.0, key.size)
    rng = np.random.default_rng(905)
    G = S.sfg_laplacian_csr(n, dev(u), dev(v), dev(w.astype(np.float32)))
    theta = dev((0.3 * rng.standard_normal(S.sfg_mpnn_param_count())).astype(np.float32))
    X, E = dev(rng.standard_normal((n, 8)).astype(np.float32)), dev(rng.standard_normal((u.size, 4)).astype(np.float32))
    want = S.sfg_mpnn_forward(G, theta, X, dev(u), dev(v), E)
    assert torch.equal(S.sfg_mpnn_forward(at_the_end(G), theta, X, dev(u), dev(v), E), want)
