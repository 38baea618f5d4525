"""The surrogate's FP32 forward, loss and gradient at the edges of their 32-row tiles and workgroup strides, against
the FP64 reference; FP32 inference and a node feature block that is not 16-byte aligned give the same predictions."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import mpnn as M

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# nodes and scored edges around one tile, one workgroup (128 rows), and more tiles than the grid takes at once
@pytest.mark.parametrize("n,ne", [(2, 1), (31, 31), (32, 32), (33, 33), (127, 129), (128, 128), (129, 160),
                                  (40000, 33000), (900, 70001)])
def test_loss_and_gradient(n, ne):
    from paper_2008_07633_amd import sfg as S

    rng = np.random.default_rng(680 + n)
    g = W.random_connected(n, 2 * ne, seed=681 + ne, wdist=("lognormal", 0.0, 1.0))
    ne = min(ne, g.m)
    cand = np.sort(rng.choice(g.m, ne, replace=False)).astype(np.int32)
    w32 = g.w.astype(np.float32)
    G = S.sfg_laplacian_csr(g.n, dev(g.u), dev(g.v), dev(w32))
    X = rng.standard_normal((g.n, 8)).astype(np.float32)
    X[:, 0] = 1.0
    E = rng.standard_normal((ne, 4)).astype(np.float32)
    y = rng.standard_normal(ne).astype(np.float32)
    theta = (M.init_params(682) + 0.02).astype(np.float32)
    A, d = M.norm_adjacency(g.n, g.u, g.v, w32.astype(np.float64))
    ref, cache = M.forward(theta.astype(np.float64), A, d, X.astype(np.float64), g.u, g.v, cand, E.astype(np.float64))
    gref = M.backward(theta.astype(np.float64), A, d, X.astype(np.float64), y.astype(np.float64), ref, cache)
    args = (G, dev(theta), dev(X), dev(g.u), dev(g.v), dev(E))
    pred, loss, grad = S.sfg_mpnn_loss_grad(*args, dev(y), cand=dev(cand))
    # the longest chain of dependent FP32 roundings of a prediction: two aggregations, 17 + 65 + 69 + 33 terms
    scale = np.abs(ref).max()
    assert np.abs(pred.cpu().numpy() - ref).max() <= 2e-5 * scale
    assert abs(loss.item() - M.loss(ref, y)) <= 1e-4 * M.loss(ref, y)
    o, gg = 0, grad.cpu().numpy()
    for name, shape in M.LAYOUT:
        c = int(np.prod(shape))
        assert np.abs(gg[o:o + c] - gref[o:o + c]).max() <= 1e-4 * max(np.abs(gref[o:o + c]).max(), 1e-12), name
        o += c
    again = S.sfg_mpnn_loss_grad(*args, dev(y), cand=dev(cand))
    assert all(torch.equal(a, b) for a, b in zip((pred, loss, grad), again))      # no order of scheduling in them
    shifted = torch.empty(g.n * 8 + 1, dtype=torch.float32, device="cuda")[1:].reshape(g.n, 8).copy_(dev(X))
    for nf in (args[2], shifted):
        inf = S.sfg_mpnn_forward(G, args[1], nf, *args[3:5], args[5], cand=dev(cand), act=torch.float32)
        assert torch.equal(inf, pred)
