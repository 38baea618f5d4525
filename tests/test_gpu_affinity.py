"""sfg_affinity's lane-group kernel (rows of 32 to 256 bytes) against the one-lane-per-edge kernel, which a block
whose start is not 16-byte aligned takes: both add every sum in column order, so the bits agree."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,k", [(torch.float32, 8), (torch.float32, 16), (torch.float32, 32), (torch.float32, 64),
                                     (torch.float64, 4), (torch.float64, 8), (torch.float64, 16),
                                     (torch.float64, 32)])
@pytest.mark.parametrize("extra", [1, 4000])
def test_affinity_groups_add_in_column_order(dtype, k, extra):
    from paper_2008_07633_amd import sfg as S

    g = W.random_connected(65 if extra == 1 else 3001, extra, seed=600 + k)      # 65 edges: a ragged last workgroup
    u, v = torch.from_numpy(g.u).cuda(), torch.from_numpy(g.v).cuda()
    x = torch.from_numpy(W.random_block(g.n, k, 601)).to(dtype).cuda()
    x[3] = 0.0                                                                     # (centred: not a zero row)
    shifted = torch.empty(g.n * k + 1, dtype=dtype, device="cuda")[1:].reshape(g.n, k).copy_(x)
    assert x.data_ptr() % 16 == 0 and shifted.data_ptr() % 16 != 0
    got, ref = S.sfg_affinity(x, u, v), S.sfg_affinity(shifted, u, v)
    assert torch.equal(got, ref)
    xb = x.double().cpu().numpy()
    xb = xb - xb.mean(0)
    d = (xb[g.u] * xb[g.v]).sum(1) ** 2 / ((xb[g.u] ** 2).sum(1) * (xb[g.v] ** 2).sum(1))
    # each of the k products and sums of a sum of terms below |xp||xq| rounds once, then two more products and a
    # quotient; the affinity is at most 1
    tol = (4 * k + 8) * (2.0 ** -24 if dtype == torch.float32 else 2.0 ** -53)
    assert np.abs(got.double().cpu().numpy() - d).max() <= tol


def test_affinity_of_a_constant_block_is_zero():
    from paper_2008_07633_amd import sfg as S

    g = W.grid2d(5, 7, seed=602)
    x = torch.full((g.n, 16), 0.25, device="cuda")
    aff = S.sfg_affinity(x, torch.from_numpy(g.u).cuda(), torch.from_numpy(g.v).cuda())
    assert bool((aff == 0).all())
