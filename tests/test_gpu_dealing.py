"""Sweeps on dense graphs whose rows are dealt to the XCDs in contiguous ranges or, where one range would hold too many
of the entries, in chunks: the same values for a node whatever its number."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def dense_graph(n, rng):
    """About 12 edges a node, ends drawn with density ~ i^(-1/2): the first ids hold most of the entries."""
    a, b = (np.minimum((n * rng.random(12 * n) ** 2).astype(np.int64), n - 1) for _ in range(2))
    a, b = np.r_[a, np.arange(1, n)], np.r_[b, np.arange(n - 1)]
    return np.unique(np.minimum(a, b) * n + np.maximum(a, b))


# rows that fill whole rounds of chunks and a rest, and fewer than one round
@pytest.mark.parametrize("n", [3000, 70001])
@pytest.mark.parametrize("dt,k,tol", [(torch.float64, 16, 1e-12), (torch.float32, 16, 1e-4), (torch.float32, 5, 1e-4)])
def test_numbering(n, dt, k, tol):
    from paper_2008_07633_amd import sfg as S

    rng = np.random.default_rng(950 + n)
    key = dense_graph(n, rng)
    key = key[key // n != key % n]
    u, v, w = key // n, key % n, rng.uniform(0.5, 2.0, key.size)
    degree = np.bincount(np.r_[u, v], minlength=n)
    share = np.add.reduceat(degree, np.arange(8) * n // 8)
    assert share.max() > 1.5 * share.mean() and degree.mean() >= 8
    x0, out = rng.standard_normal((n, k)), []
    for ids in (np.arange(n), rng.permutation(n)):
        a, b = ids[u], ids[v]
        o = np.argsort(np.minimum(a, b) * n + np.maximum(a, b))
        G = S.sfg_laplacian_csr(n, dev(np.minimum(a, b)[o].astype(np.int32)), dev(np.maximum(a, b)[o].astype(np.int32)),
                                dev(w[o]).to(dt))
        X0 = np.empty_like(x0)
        X0[ids] = x0
        out.append(S.sfg_smooth(G, dev(X0), 4, storage=dt).cpu().numpy()[ids])
    # rows of some hundred entries, added in another order, over four sweeps
    assert np.abs(out[0] - out[1]).max() <= tol * np.abs(out[1]).max()
