"""Row pointers (an exclusive scan over the nodes) around the sizes at which the scan takes another number of launches:
one tile of 2048, four tiles, 2048 tiles."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 2047, 2048, 2049, 6143, 8191, 8192, 8193, 100000, 4194303, 4194304, 4194305])
def test_row_pointers(n):
    from paper_2008_07633_amd import sfg as S

    rng = np.random.default_rng(740)
    a = np.arange(n - 1)
    on = rng.random(n - 1) < 0.7                # a path with gaps: rows of 0, 1 and 2 entries
    on[0] = True
    u, v = a[on].astype(np.int32), (a[on] + 1).astype(np.int32)
    G = S.sfg_laplacian_csr(n, torch.from_numpy(u).cuda(), torch.from_numpy(v).cuda(),
                            torch.ones(u.size, dtype=torch.float64, device="cuda"))
    deg = np.bincount(u, minlength=n) + np.bincount(v, minlength=n)
    assert np.array_equal(G.rowptr.cpu().numpy(), np.r_[0, np.cumsum(deg)])
