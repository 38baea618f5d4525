"""A call that fails on its scores leaves the caller's mask as it was."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# selections by one workgroup (up to 16,384 candidates) and by passes
@pytest.mark.parametrize("side", [40, 200])
@pytest.mark.parametrize("kw", [dict(), dict(storage=torch.float32), dict(levels=2),
                                dict(storage=torch.float16, final_f32=True, band=0.01)])
def test_keep_after_nan(side, kw):
    from paper_2008_07633_amd import sfg as S

    g = W.grid2d(side, side, seed=920)
    blocks = kw.get("levels", 1)
    x0 = np.random.default_rng(921).standard_normal((blocks, g.n, 4))
    x0[0, g.n // 2, 1] = np.nan
    keep = torch.full((g.m,), 77, dtype=torch.uint8, device="cuda")
    with pytest.raises(S.SfgError, match="SFG_ENUMERIC"):
        S.sfg_sparsify(g.n, dev(g.u), dev(g.v), dev(g.w), dev(x0), S.make_params(k=4, sweeps=3, **kw), keep=keep)
    assert bool((keep == 77).all())
