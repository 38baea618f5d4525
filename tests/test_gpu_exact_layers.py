"""The surrogate's layers and head on small whole numbers and degrees that are powers of two: every FP32 sum is exact,
so the predictions have to equal a reference that rounds to BF16 where the kernels do (and nowhere in FP32) -- with one
row of inputs of a layer or of the head at a time, with all of them, and with a hub row.  And the aggregate's quotients
at the smallest numbers, where their remainders cannot be held: as a division rounds them."""
import numpy as np
import pytest
import torch

import workloads as W
from oracle import mpnn as M

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def bf(x):
    """FP32 values rounded to BF16, to nearest even."""
    return torch.from_numpy(np.asarray(x, dtype=np.float32)).bfloat16().double().numpy()


def product(x, w, b=0.0):
    """x @ w + b, if an FP32 sum of its terms is exact in any order: their magnitudes add up to less than 2^24 times the
    power of two that all of them are multiples of."""
    terms = np.r_[np.outer(np.unique(np.abs(x)), np.unique(np.abs(w))).ravel(), np.ravel(b)]
    unit = 2.0 ** -40
    while unit < 1 and not (terms % (2 * unit)).any():
        unit *= 2
    assert (np.abs(x) @ np.abs(w) + np.abs(b)).max(initial=0.0) < 2 ** 24 * unit
    return x @ w + b


def reference(theta, A, d, X, u, v, cand, E, act):
    r = bf if act == torch.bfloat16 else np.asarray
    p = {k: r(x) if k not in ("bh1", "wh2", "bh2") else x for k, x in M.unpack(theta).items()}

    def layer(x, ws, wn, b):
        mean = r(product(A.toarray(), x) / d[:, None])
        return r(np.maximum(product(np.hstack([r(x), mean]), np.vstack([ws, wn]), b), 0.0))

    h = layer(layer(X, p["Ws1"], p["Wn1"], p["b1"]), p["Ws2"], p["Wn2"], p["b2"])
    hp, hq = h[u[cand]], h[v[cand]]
    z = np.concatenate([r(np.abs(hp - hq)), r(hp * hq), r(E)], axis=1)
    return product(np.maximum(product(z, p["Wh1"], p["bh1"]), 0.0), p["wh2"], p["bh2"])


def graph(n, per, hub, rng):
    g = W.random_connected(n, int(per * n), seed=930 + n + int(10 * per))
    key = g.u.astype(np.int64) * n + g.v
    if hub:
        far = np.setdiff1d(np.arange(n), [n // 2])
        key = np.unique(np.r_[key, np.minimum(far, n // 2) * n + np.maximum(far, n // 2)])
    return (key // n).astype(np.int32), (key % n).astype(np.int32)


def parameters(which, row, rng):
    """Whole weights: all of them (sparse), or pass-through layers and one input row of `which`."""
    p = {k: np.zeros(s) for k, s in M.LAYOUT}
    sign = lambda *s: rng.choice([-1.0, 1.0], s)      # noqa: E731
    p["wh2"], p["bh2"] = rng.integers(-100, 101, 32).astype(float), np.array([3.0])
    if which == "all":
        for k, s in M.LAYOUT[:6]:
            p[k] = rng.choice([-1.0, 1.0], s) * (rng.random(s) < (0.15 if len(s) == 1 or s[0] == 8 else 0.04))
        p["Wh1"], p["bh1"] = sign(68, 32) * (rng.random((68, 32)) < 0.1), rng.integers(-2, 3, 32).astype(float)
        p["wh2"] = rng.integers(-4, 5, 32).astype(float)
        return M.pack(p)
    p["Ws1"] = np.eye(8)[np.arange(32) % 8].T * sign(32)           # hidden j: feature j % 8, one sign
    p["Ws2"] = np.eye(32)
    p["Wh1"][:32] = np.eye(32)                                     # |hp - hq| through to the last layer
    if which == "layer 1":
        p["Ws1"] = np.zeros((8, 32))
        rows = [p["Ws1"][i] for i in range(8)] + [p["Wn1"][i] for i in range(8)] + [p["b1"]]
        rows[row][:] = sign(32)
    elif which == "layer 2":
        p["Ws2"] = np.zeros((32, 32))
        rows = [p["Ws2"][i] for i in range(32)] + [p["Wn2"][i] for i in range(32)] + [p["b2"]]
        rows[row][:] = sign(32)
        p["b2"] += 2.0 * (row < 64)
    else:
        p["Wh1"][:] = 0.0
        rows = [p["Wh1"][i] for i in range(68)] + [p["bh1"]]
        rows[row][:] = sign(32)
        p["bh1"] += 1.0
    return M.pack(p)


# entries per node: below 4, to 6, above (three forms of the layers), and a hub row beside the widest
@pytest.mark.parametrize("act", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n,per,hub", [(150, 0.3, False), (150, 1.8, False), (150, 5, False), (200, 5, True),
                                       (65, 0.3, True)])
def test_whole_numbers(n, per, hub, act):
    from paper_2008_07633_amd import sfg as S

    rng = np.random.default_rng(931 + n)
    u, v = graph(n, per, hub, rng)
    A, _ = M.norm_adjacency(n, u, v, np.ones(u.size))
    d = np.exp2(rng.integers(0, 3, n))
    G = S.sfg_laplacian_csr(n, dev(u), dev(v), dev(np.ones(u.size, np.float32)))
    G.deg = dev(d.astype(np.float32))
    cand = np.sort(rng.choice(u.size, u.size - u.size // 5, replace=False)).astype(np.int32)
    X0, E = rng.integers(-2, 3, (n, 8)).astype(np.float32), rng.integers(-9, 10, (cand.size, 4)).astype(np.float32)
    for which, rows in (("all", 3), ("layer 1", 17), ("layer 2", 65), ("head", 69)):
        if which == "all" and hub:
            continue       # the hub's sums times each other are no longer exact
        for row in range(rows):
            theta = parameters(which, row, rng)
            X = np.sign(X0) if which == "all" else X0
            want = reference(theta, A, d, X.astype(np.float64), u, v, cand, E.astype(np.float64), act)
            got = S.sfg_mpnn_forward(G, dev(theta.astype(np.float32)), dev(X), dev(u), dev(v), dev(E), cand=dev(cand),
                                     act=act)
            assert np.array_equal(got.cpu().numpy(), want.astype(np.float32)), (which, row)


def test_smallest_quotients():
    # pairs of nodes: the even one's aggregate is its neighbour's x over its degree, at 2^-124 to 2^-106 and beside
    # the midpoints of BF16, where an ulp of FP32 decides the rounding
    from paper_2008_07633_amd import sfg as S

    pairs, rng = 40000, np.random.default_rng(940)
    n = 2 * pairs
    u, v = np.arange(0, n, 2, dtype=np.int32), np.arange(1, n, 2, dtype=np.int32)
    d = (rng.uniform(1.0, 2.0, n) * np.exp2(rng.integers(0, 12, n))).astype(np.float32)
    mid = ((rng.integers(3, 22, (pairs, 8)) << 23) | (rng.integers(0, 128, (pairs, 8)) << 16) | 0x8000)
    mid = mid.astype(np.uint32).view(np.float32)
    x = (mid.astype(np.float64) * d[0::2, None]).astype(np.float32)
    x = (x.view(np.uint32) + rng.integers(0, 3, x.shape).astype(np.uint32)).view(np.float32)
    X = np.zeros((n, 8), np.float32)
    X[1::2] = x
    want = bf(x / d[0::2, None]) * 2.0 ** 100
    G = S.sfg_laplacian_csr(n, dev(u), dev(v), dev(np.ones(pairs, np.float32)))
    G.deg = dev(d)
    E = torch.zeros((pairs, 4), device="cuda")
    for c in range(8):
        p = {k: np.zeros(s) for k, s in M.LAYOUT}
        p["Wn1"][c, c], p["Ws2"][c, c], p["Wh1"][c, c], p["wh2"][c] = 2.0 ** 100, 1.0, 1.0, 1.0
        got = S.sfg_mpnn_forward(G, dev(M.pack(p).astype(np.float32)), dev(X), dev(u), dev(v), E)
        assert np.array_equal(got.cpu().numpy().astype(np.float64), want[:, c]), c
