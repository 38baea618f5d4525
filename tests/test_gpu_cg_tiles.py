"""The conjugate gradients inside the condition-number estimate at the edges of their tiles (256 / k * 16 rows of the
block, as many steps of the walk), where the tile sums of the next launch are added up by its workgroups or by launches
of their own, and where r . z and p . Ap are."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def tree_plus(n, extra, rng):
    """A random recursive tree (shallow, so that the solves are short) and `extra` more edges; its tree's marks."""
    i = np.arange(1, n)
    a, b = i, rng.integers(0, i)
    p, q = rng.integers(0, n, extra), rng.integers(0, n, extra)
    ok = p != q
    lo, hi = np.minimum(np.r_[a, p[ok]], np.r_[b, q[ok]]), np.maximum(np.r_[a, p[ok]], np.r_[b, q[ok]])
    key, first = np.unique(lo.astype(np.int64) * n + hi, return_index=True)
    return (key // n).astype(np.int32), (key % n).astype(np.int32), rng.uniform(0.5, 2.0, key.size), first < n - 1


# 8 columns: tiles of 512; 1: of 4096, 1024 lanes; 7: 146 lanes, a thread short of the workgroup; 32: from 32,769 rows
# on p . Ap, r . z and both prefix sums' offsets have launches of their own, from 8,193 the walk's alone
@pytest.mark.parametrize("n,k", [(34, 32), (128, 32), (129, 32), (8200, 32), (33000, 32), (512, 8), (513, 8), (2049, 8),
                                 (4097, 1), (577, 7), (20011, 7)])
def test_estimate(orc, n, k):
    from paper_2008_07633_amd import sfg as S

    rng = np.random.default_rng(77 + n + k)
    u, v, w, tree = tree_plus(n, n // 4 + 40, rng)
    keep = tree.astype(np.uint8)
    keep[(~tree) & (rng.random(tree.size) < 0.5)] = 2
    Y0 = orc.random_block(n, k, 5, 0)
    want = orc.kappa_estimate(n, u, v, w, keep > 0, Y0, 2)
    kap, rep = S.sfg_kappa_estimate(n, dev(u), dev(v), dev(w), dev(keep), S.make_kappa_params(k=k, steps=2, tol=1e-11),
                                    y0=dev(Y0))
    assert rep["unconverged"] == 0
    # exact solves against a relative residual of 1e-11: the bound of the estimate's other tests
    assert np.allclose(rep["ritz"], want, rtol=1e-6, atol=0)
