"""Batches on the large side of the sizes at which the launches change kernels:
beyond one wave per SIMD, beyond what is resident (the queue), beyond the wide
variants.  A few dozen to a few hundred systems, repeated to the batch's size (an
odd number of them, so that a wave's lanes and groups hold every mixture), over
short intervals; every copy equals the oracle bit for bit (the kernels do the
oracle's operations in its order, with correctly rounded functions)."""
import numpy as np
import pytest

from paper_1611_02274_amd import codegen as cg
from paper_1611_02274_amd import inputs as I

from .parity import say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1611_02274_amd as rk
    return rk


def simds():
    import torch
    return 4 * torch.cuda.get_device_properties(0).multi_processor_count


def problem(rk, orc, name, n, seed):
    """(problem, oracle's problem, y0, g, atol) of n systems."""
    if name == "vdp":
        return rk.Problem.vdp(), orc.vdp(), *I.vdp_inputs(n, seed), 1e-10
    n_sp = int(name[3:].split("_")[0])
    if name.endswith("_thermal"):
        net = I.thermal_network(n_sp)
        return (rk.Problem.network_thermal(net), orc.network_thermal(net),
                *I.thermal_inputs(net, n, seed), 1e-12)
    net = I.standard_network(n_sp)
    return rk.Problem.network(net), orc.network(net), *I.kinetics_inputs(net, n, seed), 1e-12


def repeated(a, n):
    """The systems of a, repeated to n, on the GPU."""
    import torch
    d = torch.from_numpy(np.ascontiguousarray(a)).cuda()
    return d.repeat(*([1] * (d.dim() - 1)), -(-n // d.shape[-1]))[..., :n].contiguous()


def assert_copies(got, want, label):
    """Every copy has the bits of want (NaN of any payload equal NaN)."""
    import torch
    want = repeated(want, got.shape[-1])
    same = got == want
    if got.dtype == torch.float64:
        same = torch.where(torch.isnan(want), torch.isnan(got),
                           got.view(torch.int64) == want.view(torch.int64))
    assert bool(same.all()), (label, int((~same).sum()))


def check(rk, orc, name, method, base, n, t1, rtol=1e-8, seed=51, carry=False, nan=False,
          stages=0, **opts):
    import torch
    say(f"case large {name} {method} n={n} of {base} t1={t1} rtol={rtol} carry={carry} {opts}")
    prob, pb, y0, g, atol = problem(rk, orc, name, base, seed)
    if nan:
        y0[3, 5] = np.nan
    fg = rk.integrate_rkck if method == "rkck" else rk.integrate_rkc
    y, gd = repeated(y0, n), repeated(g, n)
    if carry:
        cg_ = torch.zeros((rk.carry_rows(prob), n), dtype=torch.float64, device="cuda")
        co = orc.carry_init(pb, base)
        fo = orc.rkck_batch_carry if method == "rkck" else orc.rkc_batch_carry
        for k in range(2):
            y, st, stats = fg(prob, y, gd, k * t1, (k + 1) * t1, rtol, atol, carry=cg_, **opts)
            y0, so, sto = fo(pb, y0, g, co, k * t1, (k + 1) * t1, rtol, atol)
    else:
        y, st, stats = fg(prob, y, gd, 0.0, t1, rtol, atol, out=y, **opts)   # in place
        y0, so, sto = (orc.rkck_batch if method == "rkck" else orc.rkc_batch)(
            pb, y0, g, 0.0, t1, rtol, atol)
    torch.cuda.synchronize()
    assert sto[5].max() > stages
    assert_copies(st, so, "status")
    assert_copies(stats, sto, "stats")
    assert_copies(y, y0, "y")
    if carry:
        rows = slice(None) if method == "rkc" else slice(0, 2)
        assert_copies(cg_[rows].contiguous(), np.ascontiguousarray(co[rows]), "carry")


# more systems than eight waves of 64 on every SIMD: lanes take from the queue
@pytest.mark.parametrize("name,method,t1,opts", [
    ("vdp", "rkck", 0.5, dict(schedule=2)),
    ("vdp", "rkck", 0.2, dict(schedule=0, carry=True)),
    ("vdp", "rkc", 0.1, dict(schedule=2, refill=1, cost_order=1)),
    ("net9", "rkc", 2e-8, dict(schedule=2, carry=True, cost_order=1)),
    ("net13", "rkc", 2e-8, dict(schedule=2)),
    ("net13", "rkc", 2e-8, dict(schedule=0, refill=64, carry=True)),
    ("net13", "rkck", 5e-9, dict(schedule=2, cost_order=1)),
    ("net9_thermal", "rkck", 2e-9, dict(schedule=2)),
    ("net13_thermal", "rkc", 2e-9, dict(schedule=2, cost_order=1)),
    ("net13_thermal", "rkc", 2e-9, dict(schedule=0, carry=True)),
    # the plain kernels of more than one wave per SIMD
    ("net9", "rkck", 5e-9, dict(schedule=1)),
    ("net13_thermal", "rkck", 2e-9, dict(schedule=1, cost_order=1))])
def test_queue(rk, orc, name, method, t1, opts):
    check(rk, orc, name, method, 509, 8 * 64 * simds() + 65, t1, **opts)


# systems per wave of the networks' small batches, n / compute units: the first
# wave of two, 63 with a last wave part full, 64, and one system in a last wave
@pytest.mark.parametrize("name,method,t1", [("net9", "rkc", 2e-8), ("net13", "rkck", 5e-9),
                                            ("net13_thermal", "rkc", 2e-9)])
@pytest.mark.parametrize("per_cu,more", [(2, -1), (2, 0), (64, -1), (64, 1)])
def test_spread_edges(rk, orc, name, method, t1, per_cu, more):
    check(rk, orc, name, method, 67, per_cu * simds() // 4 + more, t1, schedule=1)


# the kernels of more than one wave per SIMD; below, reverse sweeps of 48 systems per
# wave (columns of a wave in two of the workspace's blocks) and 16, few systems
@pytest.mark.parametrize("n_sp,method,per_simd", [
    (9, "rkc", 64), (9, "rkck", 64), (13, "rkc", 64), (13, "rkck", 64),
    (9, "rkc", 10), (9, "rkck", 10), (13, "rkc", 10), (13, "rkck", 10),
    (9, "rkc", 1), (13, "rkck", 1), (9, "rkck", 0), (13, "rkc", 0)])
def test_adjoint(rk, orc, n_sp, method, per_simd):
    import torch
    base, n = 131, per_simd * simds() + 67
    say(f"case large adjoint {n_sp} {method} n={n}")
    prob, pb, y0, g, atol = problem(rk, orc, f"net{n_sp}", base, 61)
    w = I.adjoint_weights(n_sp, base, 61)
    t1 = 2e-8
    taped = rk.integrate_rkck_taped if method == "rkck" else rk.integrate_rkc_taped
    gd = repeated(g, n)
    y1, st, stats, tape = taped(prob, repeated(y0, n), gd, 0.0, t1, 1e-8, atol, max_accepted=4096,
                                ckpt_every=8)
    dy0, dth, ast = (rk.adjoint_rkck if method == "rkck" else rk.adjoint_rkc)(prob, gd, tape,
                                                                            repeated(w, n))
    torch.cuda.synchronize()
    yo, d0, dt, so = (orc.rkck_adjoint_batch if method == "rkck" else orc.rkc_adjoint_batch)(
        pb, y0, g, w, 0.0, t1, 1e-8, atol)
    assert bool((ast == 0).all()) and torch.equal(tape.count, stats[0])
    for got, want, label in ((st, so, "status"), (y1, yo, "y1"), (dy0, d0, "dy0"),
                             (dth, dt, "dlnA")):
        assert_copies(got, want, label)


# one system more than the wide variants run: the group kernels alone, with every
# wait for the other groups of a wave, carried state, the cost order, steps of more
# stages than the coefficient table holds and NaN input
@pytest.mark.parametrize("name,method,base,t1,opts", [
    ("net53", "rkc", 67, 3e-8, {}),
    ("net53", "rkc", 67, 2e-8, dict(group_align=-1, schedule=3)),
    ("net53", "rkc", 67, 2e-8, dict(group_align=8, refill=32, schedule=3)),
    ("net53", "rkc", 67, 1e-8, dict(carry=True, cost_order=1)),
    ("net53", "rkc", 24, 1e-5, dict(rtol=1e-3, nan=True, stages=32, seed=41)),
    ("net53", "rkck", 67, 1e-9, {}),
    ("net53", "rkck", 67, 5e-10, dict(carry=True, schedule=3)),
    ("net53", "rkck", 67, 5e-10, dict(nan=True, cost_order=1)),
    ("net32", "rkc", 67, 3e-8, dict(group_align=8)),
    ("net32", "rkc", 67, 1e-8, dict(carry=True, group_align=-1)),
    ("net32", "rkc", 24, 1e-5, dict(rtol=1e-3, nan=True, stages=32, seed=41)),
    ("net32", "rkck", 67, 1e-9, {}),
    ("net32", "rkck", 67, 1e-9, dict(schedule=3, refill=1, cost_order=1)),
    ("net32", "rkck", 67, 5e-10, dict(carry=True, nan=True)),
    ("net53_thermal", "rkc", 67, 1e-10, dict(cost_order=1)),
    ("net53_thermal", "rkc", 67, 1e-10, dict(carry=True, group_align=8)),
    ("net53_thermal", "rkck", 67, 2e-10, dict(nan=True)),
    ("net32_thermal", "rkc", 67, 2e-10, dict(nan=True, group_align=-1)),
    ("net32_thermal", "rkck", 67, 5e-10, dict(carry=True))])
def test_group_kernels(rk, orc, name, method, base, t1, opts):
    limit = cg.wide_limit(int(name[3:5]), name.endswith("_thermal"), method)
    check(rk, orc, name, method, base, limit * simds() + 1, t1, **opts)


@pytest.mark.parametrize("order", [[3, 2, 1, 0], [2, 0, 3, 1]])
def test_batch_order(rk, order):
    """A ragged batch's networks taken in other orders than the default."""
    import torch
    say(f"case batch order {order}")
    _, per_net = I.ragged_inputs(2000, 9, (800.0, 3000.0))
    batch = rk.Batch([rk.Problem.network(I.standard_network(k)) for k in (9, 13, 32, 53)])
    got = []
    for kw in ({}, dict(order=order)):
        ys = [torch.from_numpy(y).cuda() for y, _ in per_net]
        gs = [torch.from_numpy(g).cuda() for _, g in per_net]
        st = [torch.empty(y.shape[1], dtype=torch.int32, device="cuda") for y in ys]
        stats = [torch.empty((rk.RK_NSTATS, y.shape[1]), dtype=torch.int32, device="cuda")
                 for y in ys]
        batch.integrate_rkc(ys, gs, 0.0, 2e-7, 2, 1e-8, 1e-12, status=st, stats=stats, **kw)
        torch.cuda.synchronize()
        got.append([y.view(torch.int64) for y in ys] + st + stats)
    for a, b in zip(*got):
        assert torch.equal(a, b)
