"""The seven-body problem on lane groups: sizes around a wave's eight systems,
coincident and non-finite bodies (a body's own term is a zero times a zero kept
beside the pair values), against the oracle bit for bit."""
import numpy as np
import pytest

from paper_1611_02274_amd import inputs as I

from .parity import say


@pytest.mark.gpu
@pytest.mark.parametrize("method,n", [("rkck", 1), ("rkck", 7), ("rkck", 9), ("rkck", 24577),
                                      ("rkc", 9)])
def test_pleiades_group_equals_oracle(orc, method, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1611_02274_amd as rk
    say(f"case pleiades group {method} n={n}")
    y0 = I.pleiades_inputs(n, 61)[0].copy()
    if n == 9:
        y0[2, 1] = np.nan                            # a position
        y0[9, 2] = np.inf
        y0[17, 3] = np.nan                           # a velocity
        y0[1, 4], y0[8, 4] = y0[0, 4], y0[7, 4]      # two bodies in one place
    t1 = 0.05 if method == "rkck" else 0.005
    fn = rk.integrate_rkck if method == "rkck" else rk.integrate_rkc
    y1, st, stats = fn(rk.Problem.pleiades(), torch.from_numpy(y0).cuda(), None, 0.0, t1, 1e-8,
                       0.0)
    torch.cuda.synchronize()
    idx = np.unique(np.linspace(0, n - 1, min(n, 300)).astype(np.int64))
    yo, so, sto = (orc.rkck_batch if method == "rkck" else orc.rkc_batch)(
        orc.pleiades(), np.ascontiguousarray(y0[:, idx]), None, 0.0, t1, 1e-8, 0.0)
    y1, st, stats = y1.cpu().numpy(), st.cpu().numpy(), stats.cpu().numpy()
    assert np.array_equal(st[idx], so) and np.array_equal(stats[:, idx], sto)
    assert np.array_equal(y1[:, idx], yo, equal_nan=True)
