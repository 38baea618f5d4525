"""Calls on shapes that a kernel's usual case does not cover take times of the usual order: hub rows that share one
workgroup's nodes in a tree's layout, chains of hooks as long as the graph in the spanning forest; and the sweeps of
graphs without hub rows do not pay for the code that takes them."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def canonical(n, a, b):
    """(u, v) in order, and the place of every given edge in it."""
    key = np.minimum(a, b).astype(np.int64) * n + np.maximum(a, b)
    o = np.argsort(key)
    return (key[o] // n).astype(np.int32), (key[o] % n).astype(np.int32), o


def micros(f):
    """The shortest of five calls after two."""
    out = []
    for i in range(7):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        out.append(1e3 * a.elapsed_time(b))
    return min(out[2:])


def test_layout_of_hub_rows():
    # 256 hubs with the last ids (one workgroup of nodes), the other nodes on their rows: against a tree of random
    # parents.  One workgroup took the hubs' arcs in 4,096 steps of dependent reads, several times all of the rest.
    from paper_2008_07633_amd import sfg as S

    n, rng = 1 << 20, np.random.default_rng(910)
    i = np.arange(1, n)
    random, ids = rng.integers(0, i), rng.permutation(n)
    leaf = np.arange(n - 256)
    hubs = (np.r_[leaf, np.arange(n - 256, n - 1)],
            np.r_[n - 256 + rng.integers(0, 256, n - 256), np.arange(n - 255, n)])
    w, keep, t = dev(np.ones(n - 1)), torch.ones(n - 1, dtype=torch.uint8, device="cuda"), {}
    for name, (a, b) in {"random": (ids[i], ids[random]), "hubs": hubs}.items():
        u, v, _ = canonical(n, a, b)
        u, v = dev(u), dev(v)
        t[name] = micros(lambda: S.sfg_tree_order(n, u, v, w, keep))
    assert t["hubs"] <= 2.0 * t["random"], t


@pytest.mark.parametrize("n", [200000, 400000, 500000, 1000000])
def test_forest_of_one_chain(n):
    # a path of shuffled ids: weights rising along it (every node hooks onto the next: one chain) against random ones
    from paper_2008_07633_amd import sfg as S

    rng = np.random.default_rng(911)
    ids, t = rng.permutation(n), {}
    u, v, o = canonical(n, ids[:-1], ids[1:])
    for name, w in {"chain": (1.0 + o / n), "random": rng.uniform(1.0, 2.0, n - 1)}.items():
        a = (n, dev(u), dev(v), dev(w))
        tree, comps = S.sfg_spanning_tree(*a)
        assert comps == 1 and int(tree.sum()) == n - 1
        t[name] = micros(lambda: S.sfg_spanning_tree(*a))
    assert t["chain"] <= 3.0 * t["random"], t


def test_sweeps_without_hub_rows():
    # 32 FP32 vectors and 16 FP64 ones are as many bytes; with the hub rows' registers in every row's way the FP32
    # sweeps, which move less for the graph, took 1.18 times as long
    import workloads as W
    from paper_2008_07633_amd import sfg as S

    g, t = W.mesh3d(80, 80, 80, seed=912), {}
    for dt, k in ((torch.float32, 32), (torch.float64, 16)):
        G = S.sfg_laplacian_csr(g.n, dev(g.u), dev(g.v), dev(g.w).to(dt))
        x0 = dev(np.random.default_rng(913).standard_normal((g.n, k)))
        out = torch.empty((g.n, k), dtype=dt, device="cuda")
        t[dt] = micros(lambda: S.sfg_smooth(G, x0, 20, storage=dt, out=out))
    assert t[torch.float32] <= 1.1 * t[torch.float64], t


def test_tree_csr_of_a_dense_list():
    # the few edges that a spanning tree's mask leaves of a long list: sorting the list by digits took 0.83 of the whole
    # list's time
    import workloads as W
    from paper_2008_07633_amd import sfg as S

    g, t = W.chung_lu(50000, 500000, 2.2, seed=914), {}
    assert g.m > 8 * g.n and g.m >= 1 << 18
    u, v, w = dev(g.u), dev(g.v), dev(g.w)
    tree, _ = S.sfg_spanning_tree(g.n, u, v, w)
    ws = torch.empty(S.sfg_workspace_bytes(S.OP_LAPLACIAN_CSR, g.n, g.m, 0, w.dtype), dtype=torch.uint8, device="cuda")
    for name, mask, nnz in (("all", None, 2 * g.m), ("tree", tree, 2 * (g.n - 1))):
        out = S.sfg_laplacian_csr(g.n, u, v, w, mask=mask)
        t[name] = micros(lambda: S.sfg_laplacian_csr(g.n, u, v, w, mask=mask, ws=ws, out=out, nnz=nnz))
    assert t["tree"] <= 0.7 * t["all"], t
