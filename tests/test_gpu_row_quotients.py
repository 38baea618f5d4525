"""The passes through LDS take a row's quotients with one reciprocal where its sums and degree are of middling size, and
divide elsewhere: bit for bit what sfg_smooth's divisions give, on weights and blocks on both sides of that bound."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# powers of two that the weights and the block's columns spread over, below and above the bounds (2^40, 2^300)
@pytest.mark.parametrize("storage,wide", [(torch.float32, 0), (torch.float32, 25), (torch.float32, 45),
                                          (torch.float16, 45), (torch.float64, 0), (torch.float64, 200),
                                          (torch.float64, 340)])
@pytest.mark.parametrize("k", [4, 8, 16])
def test_same_bits(storage, wide, k, monkeypatch):
    from paper_2008_07633_amd import sfg as S

    monkeypatch.setenv("SFG_SWEEP_HOPS", "2" if storage == torch.float64 else "3")
    g = W.powergrid(40, 37, 0.02, seed=720)
    rng = np.random.default_rng(721 + wide + k)
    w = rng.uniform(0.5, 2.0, g.m) * np.exp2(rng.integers(-wide, wide + 1, g.m))
    u, v = dev(g.u), dev(g.v)
    tree, _ = S.sfg_spanning_tree(g.n, u, v, dev(w))
    order = S.sfg_tree_order(g.n, u, v, dev(w), tree).order
    H = S.sfg_laplacian_csr(g.n, u, v, dev(w).to(torch.float64 if storage == torch.float64 else torch.float32),
                            mask=tree)
    X0 = W.random_block(g.n, k, 722)
    X0 = X0 * (np.exp2(rng.integers(-wide, wide + 1, k)) if storage != torch.float16 else 1.0)
    X0[:, 1] = 0.0                                  # sums of zero
    X0[: g.n // 2, 2] = 0.0
    X0 = dev(X0)
    for sweeps in (5, 12):
        info = {}
        got = S.sfg_smooth_ordered(H, order, X0, sweeps, 0.5, storage=storage, info=info)
        ref = S.sfg_smooth(H, X0, sweeps, 0.5, storage=storage)
        bits = {8: torch.int64, 4: torch.int32, 2: torch.int16}[got.element_size()]
        assert torch.equal(got.isnan(), ref.isnan())
        assert torch.equal(got.view(bits)[~ref.isnan()], ref.view(bits)[~ref.isnan()]), (sweeps, info)
        assert info["sweeps_per_pass"] > 1
