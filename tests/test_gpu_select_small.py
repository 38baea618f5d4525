"""Top-k selection by one workgroup (up to 16,384 scores) against the oracle, up to and just past its bound: all scores
different, nearly all alike, ties at the threshold, signed values with infinities and both zeros."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.float64, torch.float32])
@pytest.mark.parametrize("ne", [1, 2, 63, 1024, 1025, 3969, 16383, 16384, 16385])
@pytest.mark.parametrize("kind", ["distinct", "alike", "ties", "signed"])
def test_select(orc, dt, ne, kind):
    from paper_2008_07633_amd import sfg as S

    rng = np.random.default_rng(730 + ne)
    s = {"distinct": lambda: rng.lognormal(0.0, 3.0, ne), "alike": lambda: np.where(rng.random(ne) < 0.01, 2.0, 1.0),
         "ties": lambda: rng.integers(0, 7, ne).astype(float),
         "signed": lambda: rng.choice(np.r_[rng.standard_normal(50), 0.0, np.inf, -np.inf], ne)}[kind]()
    s = s.astype(np.float64 if dt == torch.float64 else np.float32)
    for k in sorted({1, (ne + 9) // 10, ne // 2 + 1, ne}):
        sel, tau = S.sfg_select_topk(torch.from_numpy(s).cuda(), k)
        want, wtau = orc.select_topk(s.astype(np.float64), np.arange(ne), k)
        got = np.flatnonzero(sel.cpu().numpy())
        assert np.array_equal(got, np.sort(np.asarray(want))) and float(tau) == wtau, k
