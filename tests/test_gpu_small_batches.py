"""Small batches of the one-lane kernels, spread over the SIMDs with the other
lanes of a wave repeating its systems: sizes around the steps of the systems
per wave (1024 SIMDs), the last wave part full, in place, with the order map,
and the taped forward and reverse sweeps, against the oracle bit for bit."""
import numpy as np
import pytest

from paper_1611_02274_amd import inputs as I

from .parity import compare, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1611_02274_amd as rk
    return rk


@pytest.mark.parametrize("problem,method,n,opts", [
    ("vdp", "rkck", 1, dict(schedule=1)),
    ("vdp", "rkck", 1023, dict(schedule=2)),
    ("vdp", "rkck", 1025, dict(schedule=1)),
    ("vdp", "rkck", 3070, dict(schedule=0, cost_order=1)),
    ("vdp", "rkc", 2049, dict(schedule=0)),
    ("net9", "rkc", 5, dict(schedule=0)),
    ("net9", "rkc", 1027, dict(schedule=1, cost_order=1)),
    ("net13", "rkck", 2050, dict(schedule=2))])
def test_spread_batch(rk, orc, problem, method, n, opts):
    import torch
    say(f"case spread {method} {problem} n={n} {opts}")
    if problem == "vdp":
        y0, g = I.vdp_inputs(n, 31)
        prob, pb, t1, atol = rk.Problem.vdp(), orc.vdp(), 2.0, 1e-10
    else:
        net = I.network_of(problem)
        y0, g = I.kinetics_inputs(net, n, 32)
        prob, pb, t1, atol = rk.Problem.network(net), orc.network(net), 2e-8, 1e-12
    fn = rk.integrate_rkck if method == "rkck" else rk.integrate_rkc
    yd, gd = torch.from_numpy(y0).cuda(), torch.from_numpy(g).cuda()
    _, st, stats = fn(prob, yd, gd, 0.0, t1, 1e-8, atol, out=yd, **opts)
    torch.cuda.synchronize()
    yo, so, sto = (orc.rkck_batch if method == "rkck" else orc.rkc_batch)(pb, y0, g, 0.0, t1,
                                                                         1e-8, atol)
    rep = compare(yd.cpu().numpy(), st.cpu().numpy(), stats.cpu().numpy(), yo, so, sto, atol,
                  f"spread {method}/{problem}/n={n}", count_fraction=1.0)
    assert rep["bitwise_equal"] == 1.0


@pytest.mark.parametrize("method,n", [("rkc", 3), ("rkc", 1026), ("rkck", 1026)])
def test_spread_adjoint(rk, orc, method, n):
    import torch
    say(f"case spread adjoint {method} n={n}")
    net = I.standard_network(9)
    y0, g = I.kinetics_inputs(net, n, 33)
    w = I.adjoint_weights(net.n_sp, n, 33)
    prob, pb = rk.Problem.network(net), orc.network(net)
    yd, gd, wd = (torch.from_numpy(a).cuda() for a in (y0, g, w))
    taped = rk.integrate_rkck_taped if method == "rkck" else rk.integrate_rkc_taped
    y1, st, stats, tape = taped(prob, yd, gd, 0.0, 2e-8, 1e-8, 1e-12, max_accepted=4096,
                                ckpt_every=8)
    dy0, dth, ast = (rk.adjoint_rkck if method == "rkck" else rk.adjoint_rkc)(prob, gd, tape, wd)
    torch.cuda.synchronize()
    assert np.array_equal(tape.count.cpu().numpy(), stats[0].cpu().numpy())
    yo, d0, dt, so = (orc.rkck_adjoint_batch if method == "rkck" else orc.rkc_adjoint_batch)(
        pb, y0, g, w, 0.0, 2e-8, 1e-8, 1e-12)
    assert np.all(ast.cpu().numpy() == 0) and np.array_equal(st.cpu().numpy(), so)
    assert np.array_equal(y1.cpu().numpy(), yo)
    for a, b in ((dy0, d0), (dth, dt)):
        a = a.cpu().numpy()
        # the reverse sweep's operations are the oracle's up to the order of a few sums
        assert np.abs(a - b).max() <= 1e-9 * np.abs(b).max()
