"""The energy equation on lane groups: the wide layout (one unknown per lane) is
disjoint and decodes to the reference evaluation's operands and terms; on the
GPU, sizes around the switch between the wide and the 32-lane kernels, steps of
more stages than the coefficient table holds and non-finite input, against the
oracle bit for bit."""
import numpy as np
import pytest

from paper_1611_02274_amd import codegen as cg
from paper_1611_02274_amd import inputs as I

from .parity import say


@pytest.mark.parametrize("n_sp", [32, 53])
def test_thermal_wide_layout(n_sp):
    net = I.thermal_network(n_sp)
    G = cg._wide_layout(net, 64, thermal=True)
    R = G["R"]
    areas = sorted([(0, n_sp + 2), (G["off_q"], G["off_q"] + R * 64),
                    (G["off_zero"], G["off_zero"] + 1),
                    (G["off_red"], G["off_red"] + cg.GROUP_COEF_DOUBLES),
                    (G["off_e1"], G["off_e1"] + n_sp + n_sp % 2),
                    (G["off_e2"], G["off_e2"] + n_sp + n_sp % 2),
                    (G["off_q"] + G["neg"], G["off_q"] + G["neg"] + R * 64)])
    for (_, b0), (a1, _) in zip(areas, areas[1:]):
        assert b0 <= a1
    assert areas[-1][1] <= G["lds"] and 8 * G["lds"] < 1 << 16
    assert G["off_red"] + n_sp + 1 <= G["off_q"] + G["neg"]
    assert all(G[k] % 2 == 0 for k in ("lds", "off_red", "off_e1", "off_e2"))
    seen = {j: p for p, j in enumerate(G["rx_of"]) if j >= 0}
    assert len(seen) == net.n_rx
    for j, p in seen.items():
        r, m = p % 64, p // 64
        want = [int(k) if k >= 0 else n_sp for k in (*net.reac[j], *net.prod[j])]
        assert [o // 8 for o in G["ops"][(r * R + m) * 4:(r * R + m) * 4 + 4]] == want
        assert n_sp not in want or m >= G["m_first"]
    for r in range(64):
        want = []
        for j in range(net.n_rx) if 1 <= r <= n_sp else ():
            want += [G["off_q"] + G["neg"] + seen[j] for s in net.reac[j] if int(s) == r - 1]
            want += [G["off_q"] + seen[j] for s in net.prod[j] if int(s) == r - 1]
        got = [a // 8 for a in G["tm"][r * G["T"]:(r + 1) * G["T"]]]
        assert got[:len(want)] == want
        assert all(a == G["off_zero"] for a in got[len(want):])


@pytest.mark.gpu
@pytest.mark.parametrize("n_sp,method,n,t1,rtol", [
    (53, "rkc", 1, 1e-8, 1e-8), (53, "rkc", 1024, 1e-9, 1e-8), (53, "rkc", 1025, 1e-9, 1e-8),
    (32, "rkc", 1024, 2e-9, 1e-8), (32, "rkc", 1025, 2e-9, 1e-8),
    (32, "rkck", 6145, 3e-10, 1e-8), (53, "rkck", 12289, 1e-10, 1e-8),
    (53, "rkc", 24, 3e-6, 1e-3), (32, "rkc", 24, 3e-6, 1e-3)])
def test_thermal_switch(orc, n_sp, method, n, t1, rtol):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1611_02274_amd as rk
    say(f"case thermal group net{n_sp} {method} n={n} t1={t1} rtol={rtol}")
    net = I.thermal_network(n_sp)
    y0, g = I.thermal_inputs(net, n, 51, (1000.0, 2500.0))
    if n == 24:
        y0[4, 5] = np.nan
        y0[7, 6] = np.inf
    fn = rk.integrate_rkck if method == "rkck" else rk.integrate_rkc
    y1, st, stats = fn(rk.Problem.network_thermal(net), torch.from_numpy(y0).cuda(),
                       torch.from_numpy(g).cuda(), 0.0, t1, rtol, 1e-12)
    torch.cuda.synchronize()
    # systems are independent of each other: the oracle takes a spread of the large batches
    idx = np.unique(np.linspace(0, n - 1, min(n, 300)).astype(np.int64))
    yo, so, sto = (orc.rkck_batch if method == "rkck" else orc.rkc_batch)(
        orc.network_thermal(net), np.ascontiguousarray(y0[:, idx]),
        np.ascontiguousarray(g[:, idx]), 0.0, t1, rtol, 1e-12)
    if n == 24:
        assert np.sort(sto[5])[-3] > 32, "steps of more stages than the table holds"
    y1, st, stats = y1.cpu().numpy(), st.cpu().numpy(), stats.cpu().numpy()
    assert np.array_equal(st[idx], so) and np.array_equal(stats[:, idx], sto)
    assert np.array_equal(y1[:, idx], yo, equal_nan=True)
