"""The CSR of large lists of more than 8 edges per node (lower parts from a stable sort by the larger end) against a
host build: same rows, columns, weights, ids and degrees, with and without a mask."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def edge_list(n, m, seed, hub):
    """m distinct edges of n nodes; hub = 'first' or 'last' joins that node to every other."""
    rng = np.random.default_rng(seed)
    a, b = rng.integers(0, n, 2 * m), rng.integers(0, n, 2 * m)
    key = np.unique(np.minimum(a, b)[a != b] * n + np.maximum(a, b)[a != b])
    key = rng.permutation(key)[:m - n + 1]
    star = np.arange(1, n) if hub == "first" else np.arange(n - 1) * n + n - 1
    key = np.unique(np.concatenate([key, star]))
    return (key // n).astype(np.int32), (key % n).astype(np.int32), rng.uniform(0.5, 2.0, key.size)


def host_csr(n, u, v, w, ids):
    row, col = np.r_[u, v], np.r_[v, u]
    o = np.lexsort((col, row))
    row, col, val, eid = row[o], col[o], np.r_[w, w][o], np.r_[ids, ids][o]
    # bincount adds its weights in order: each degree is the sequential sum of the row
    return np.r_[0, np.cumsum(np.bincount(row, minlength=n))], col, val, eid, \
        np.bincount(row, weights=val.astype(np.float64), minlength=n)


# two digit passes, three, and a list just over the size from which it is sorted; the last mask leaves a tree's worth
@pytest.mark.parametrize("n,m,hub", [(1500, 300000, "last"), (70000, 700000, "first"), (70000, 600001, "last"),
                                     (2000, (1 << 18) + 2100, "first")])
@pytest.mark.parametrize("share", [1.0, 0.5, 0.01])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_sorted_build_matches_host(n, m, hub, share, dtype):
    from paper_2008_07633_amd import sfg as S

    u, v, w = edge_list(n, m, 620 + n, hub)
    assert u.size > 8 * n and u.size >= 1 << 18
    mask = None if share == 1.0 else (np.random.default_rng(621).random(u.size) < share).astype(np.uint8)
    t = [torch.from_numpy(a).cuda() for a in (u, v, w)]
    wt = t[2].to(dtype)
    H = S.sfg_laplacian_csr(n, t[0], t[1], wt, mask=None if mask is None else torch.from_numpy(mask).cuda())
    ids = np.arange(u.size) if mask is None else np.flatnonzero(mask)
    ptr, col, val, eid, deg = host_csr(n, u[ids], v[ids], wt.cpu().numpy()[ids], ids)
    assert H.nnz == 2 * ids.size
    got = [x.cpu().numpy() for x in (H.rowptr, H.col[:H.nnz], H.val[:H.nnz], H.eid[:H.nnz], H.deg)]
    for a, b in zip(got, (ptr, col, val, eid, deg.astype(got[4].dtype))):
        assert np.array_equal(a, b)


def test_masked_scoring_graphs_match_oracle(orc):
    # inside a call that cannot tell how many edges its mask leaves (several rounds), the masked CSR of such a list is
    # sorted too; a caller's mask, a spanning tree as a rule, takes the edge-parallel build
    import workloads as W
    from paper_2008_07633_amd import sfg as S

    n, rounds, k, sweeps, frac = 2000, 3, 4, 4, 0.2
    u, v, w = edge_list(n, (1 << 18) + 3000, 640, "first")
    assert u.size > 8 * n and u.size >= 1 << 18
    X0s = np.stack([W.random_block(n, k, 641 + r) for r in range(rounds)])
    ref = orc.sparsify_rounds(n, u, v, w, list(X0s), rounds, sweeps, frac)
    t = [torch.from_numpy(a).cuda() for a in (u, v, w, X0s)]
    keep, _ = S.sfg_sparsify(n, *t, S.make_params(k=k, sweeps=sweeps, frac=frac, rounds=rounds))
    assert np.array_equal(keep.cpu().numpy(), ref.keep)
