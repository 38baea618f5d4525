"""Hub rows (over 256 entries) in reduced precision, for every number of lanes a row takes: two sweeps on whole numbers
and degrees that are powers of two, whose FP32 sums are exact in any order, against a reference that rounds where the
storage does."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("length", [256, 257, 1000, 4096, 4097, 20000])
@pytest.mark.parametrize("dt", [torch.float32, torch.float16, torch.bfloat16])
@pytest.mark.parametrize("k", [4, 5, 12, 13, 16, 24])
def test_two_sweeps(length, dt, k):
    from paper_2008_07633_amd import sfg as S
    import scipy.sparse as sp

    n, rng = length + 7, np.random.default_rng(960 + length + k)
    leaf = np.sort(rng.choice(n - 1, length, replace=False)) + 1      # node 0 beside them, and a path of all
    u = np.r_[np.zeros(length, int), np.arange(1, n - 1)]
    v = np.r_[leaf, np.arange(2, n)]
    w = rng.integers(1, 4, u.size).astype(np.float64)
    A = sp.coo_matrix((np.r_[w, w], (np.r_[u, v], np.r_[v, u])), shape=(n, n)).tocsr()
    d = np.exp2(rng.integers(1, 3, n))
    d[0] = 2.0 ** 13
    x0 = np.zeros((n, k))                                               # columns of -1, 0 and 1 with sum 0
    for c in range(k):
        at = rng.permutation(n)
        x0[at[:n // 3], c], x0[at[n // 3:2 * (n // 3)], c] = 1.0, -1.0

    def sweep(x):
        # the hub's sum is one of multiples of 1/8, the others', of a few terms, of multiples of 2^-18
        assert not (x[1:] % 2.0 ** -3).any() and (abs(A)[0] @ np.abs(x)).max() < 2 ** 21
        assert not (x % 2.0 ** -18).any() and (abs(A)[1:] @ np.abs(x)).max() < 2 ** 6
        y = 0.5 * x + 0.5 * (A @ x) / d[:, None]
        assert np.array_equal(y.astype(np.float32), y)
        return y

    y1 = sweep(x0)
    want = sweep(torch.from_numpy(y1).to(dt).double().numpy())
    G = S.sfg_laplacian_csr(n, dev(u.astype(np.int32)), dev(v.astype(np.int32)), dev(w.astype(np.float32)))
    G.deg = dev(d.astype(np.float32))
    got = S.sfg_smooth(G, dev(x0), 2, 0.5, storage=dt, final_f32=dt != torch.float32)
    assert np.array_equal(got.cpu().numpy().astype(np.float64), want)
