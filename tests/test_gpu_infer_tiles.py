"""BF16 inference at the edges of its 16-row tiles and workgroups, below and above the density from which more entries
are in flight per row, with a hub row, against the FP64 reference."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import mpnn as M

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# nodes and scored edges around one tile (16), one workgroup (64), more tiles than the grid takes at once (131,072);
# edges per node: 2 and 3 are the sparse form, 6 the dense one
@pytest.mark.parametrize("n,per,ne", [(2, 1, 1), (15, 2, 15), (16, 2, 16), (17, 2, 17), (63, 6, 65), (64, 6, 64),
                                      (65, 6, 100), (3000, 6, 9000), (140000, 2, 139000)])
def test_predictions(n, per, ne):
    from paper_2008_07633_amd import sfg as S

    rng = np.random.default_rng(700 + n)
    g = W.random_connected(n, per * n, seed=701 + n, wdist=("lognormal", 0.0, 1.0))
    u, v, w = g.u, g.v, g.w
    if n == 3000:       # node 7 beside everyone
        key = np.unique(np.r_[u.astype(np.int64) * n + v, np.minimum(7, np.r_[0:7, 8:n]) * n
                              + np.maximum(7, np.r_[0:7, 8:n])])
        u, v, w = (key // n).astype(np.int32), (key % n).astype(np.int32), rng.lognormal(0.0, 1.0, key.size)
    ne = min(ne, u.size)
    cand = np.sort(rng.choice(u.size, ne, replace=False)).astype(np.int32)
    w32 = w.astype(np.float32)
    G = S.sfg_laplacian_csr(n, dev(u), dev(v), dev(w32))
    X = rng.standard_normal((n, 8)).astype(np.float32)
    E = rng.standard_normal((ne, 4)).astype(np.float32)
    theta = (M.init_params(702) + 0.02).astype(np.float32)
    A, d = M.norm_adjacency(n, u, v, w32.astype(np.float64))
    ref, _ = M.forward(theta.astype(np.float64), A, d, X.astype(np.float64), u, v, cand, E.astype(np.float64))
    args = (G, dev(theta), dev(X), dev(u), dev(v), dev(E))
    run = lambda nf, ef, c: S.sfg_mpnn_forward(G, args[1], nf, *args[3:5], ef, cand=c, act=torch.bfloat16)   # noqa: E731
    pred = run(args[2], args[5], dev(cand))
    # inputs, weights, both layers' outputs, the aggregate and the head's inputs are rounded to BF16 (2^-9 each, in
    # sums of up to 69 terms): the bound of the BF16 check in test_gpu_surrogate.py
    assert np.abs(pred.cpu().numpy() - ref).max() < 3e-2 * np.abs(ref).max()
    # blocks that are not 16-byte aligned, and the candidates' own edge list in place of `cand`, change nothing
    off = [torch.empty(t.numel() + 1, dtype=torch.float32, device="cuda")[1:].reshape(t.shape).copy_(t)
           for t in (args[2], args[5])]
    assert torch.equal(run(*off, dev(cand)), pred)
    own = S.sfg_mpnn_forward(G, args[1], args[2], dev(u[cand]), dev(v[cand]), args[5], act=torch.bfloat16)
    assert torch.equal(own, pred)
