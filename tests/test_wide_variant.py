"""The wide variants of the 32/53-species networks (one species per lane, small
batches).  Host: the LDS areas are disjoint and every address decodes to the
reference evaluation's operands and terms in its order.  GPU: sizes around a
wave's systems and the switch to the group kernels, steps of more stages than
the coefficient table holds, non-finite input, the order map and the carried
state, against the oracle bit for bit."""
import numpy as np
import pytest

from paper_1611_02274_amd import codegen as cg
from paper_1611_02274_amd import inputs as I

from .parity import compare, say


@pytest.mark.parametrize("n_sp", [32, 53])
def test_wide_layout(n_sp):
    net = I.standard_network(n_sp)
    L = cg.wide_lanes(n_sp)
    G = cg._wide_layout(net, L)
    R = G["R"]
    areas = sorted([(0, n_sp + 2), (G["off_q"], G["off_q"] + R * L),
                    (G["off_zero"], G["off_zero"] + 1), (G["off_red"], G["off_red"] + n_sp),
                    (G["off_q"] + G["neg"], G["off_q"] + G["neg"] + R * L)])
    for (_, b0), (a1, _) in zip(areas, areas[1:]):
        assert b0 <= a1
    assert areas[-1][1] <= G["lds"] and G["lds"] % 2 == 0 and G["off_red"] % 2 == 0
    assert 8 * G["lds"] < 1 << 16
    # every reaction has one position, and the position's operands are its species
    seen = {}
    for p, j in enumerate(G["rx_of"]):
        if j < 0:
            continue
        assert j not in seen
        seen[j] = p
        r, m = p % L, p // L
        want = [int(k) if k >= 0 else n_sp for k in (*net.reac[j], *net.prod[j])]
        assert [o // 8 for o in G["ops"][(r * R + m) * 4:(r * R + m) * 4 + 4]] == want
        assert n_sp not in want or m >= G["m_first"]
    assert len(seen) == net.n_rx
    for k in range(n_sp):
        want = []
        for j in range(net.n_rx):
            want += [G["off_q"] + G["neg"] + seen[j] for s in net.reac[j] if int(s) == k]
            want += [G["off_q"] + seen[j] for s in net.prod[j] if int(s) == k]
        got = [a // 8 for a in G["tm"][k * G["T"]:(k + 1) * G["T"]]]
        assert got[:len(want)] == want
        assert all(a == G["off_zero"] for a in got[len(want):])


@pytest.fixture(scope="module")
def rk():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1611_02274_amd as rk
    return rk


@pytest.mark.gpu
@pytest.mark.parametrize("n_sp,method,n,t1,rtol,opts", [
    (53, "rkc", 1, 3e-8, 1e-8, {}),
    (53, "rkck", 3, 3e-8, 1e-8, {}),
    (53, "rkc", 1024, 2e-9, 1e-8, {}),
    (53, "rkc", 1025, 2e-9, 1e-8, {}),
    (32, "rkc", 3, 3e-8, 1e-8, dict(schedule=3)),
    (32, "rkck", 1025, 5e-9, 1e-8, dict(cost_order=1)),
    (32, "rkc", 6145, 1e-9, 1e-8, {}),
    (53, "rkc", 24, 1e-5, 1e-3, {}),
    (32, "rkc", 24, 1e-5, 1e-3, {})])
def test_wide_equals_oracle(rk, orc, n_sp, method, n, t1, rtol, opts):
    import torch
    say(f"case wide {n_sp} {method} n={n} t1={t1} rtol={rtol} {opts}")
    net = I.standard_network(n_sp)
    y0, g = I.kinetics_inputs(net, n, 41, (900.0, 2800.0))
    if n == 24:
        y0[3, 5] = np.nan
    yd, gd = torch.from_numpy(y0).cuda(), torch.from_numpy(g).cuda()
    fn = rk.integrate_rkck if method == "rkck" else rk.integrate_rkc
    y1, st, stats = fn(rk.Problem.network(net), yd, gd, 0.0, t1, rtol, 1e-12, **opts)
    torch.cuda.synchronize()
    yo, so, sto = (orc.rkck_batch if method == "rkck" else orc.rkc_batch)(
        orc.network(net), y0, g, 0.0, t1, rtol, 1e-12)
    if n == 24:
        assert sto[5].max() > 32, "steps of more stages than the table holds"
    y1, st, stats = y1.cpu().numpy(), st.cpu().numpy(), stats.cpu().numpy()
    assert np.array_equal(st, so) and np.array_equal(stats, sto)
    assert np.array_equal(y1, yo, equal_nan=True)


@pytest.mark.gpu
@pytest.mark.parametrize("n_sp,method", [(53, "rkc"), (53, "rkck"), (32, "rkc")])
def test_wide_carry(rk, n_sp, method):
    """Two substeps with carried state equal the one-lane kernels' bits, the
    carried array included."""
    import torch
    say(f"case wide carry {n_sp} {method}")
    net = I.standard_network(n_sp)
    y0, g = I.kinetics_inputs(net, 35, 42, (900.0, 2800.0))
    prob = rk.Problem.network(net)
    fn = rk.integrate_rkck if method == "rkck" else rk.integrate_rkc
    got = []
    for schedule in (0, 1):
        y, gd = torch.from_numpy(y0).cuda(), torch.from_numpy(g).cuda()
        carry = torch.zeros((rk.carry_rows(prob), 35), dtype=torch.float64, device="cuda")
        for k in range(2):
            y, st, stats = fn(prob, y, gd, k * 1e-8, (k + 1) * 1e-8, 1e-8, 1e-12, carry=carry,
                              schedule=schedule)
        torch.cuda.synchronize()
        rows = slice(None) if method == "rkc" else slice(0, 2)
        got.append([a.cpu().numpy() for a in (y, st, stats, carry[rows])])
    for a, b in zip(*got):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("n_sp,thermal", [(32, False), (53, False), (32, True), (53, True)])
def test_packed_group_addresses(n_sp, thermal):
    """The group kernels' packed LDS offsets name, for every lane of the wave,
    the operands and terms of its group's layout in its group's area."""
    net = I.standard_network(n_sp)
    G = cg._group_layout(net, 32 if thermal else cg.group_lanes(n_sp), thermal=thermal)
    L, R, per = G["L"], G["R"], G["lds_per_system"]
    op, op_words, tm, tm_words = cg._packed_addresses(G)
    assert op_words % 4 == 0 and tm_words % 4 == 0
    assert sorted(j for j in G["rx_of"] if j >= 0) == list(range(net.n_rx))

    def entry(table, words, lane, k):
        return table[lane * words + k // 2] >> (16 * (k % 2)) & 0xffff

    for lane in range(64):
        r, area = lane % L, lane // L * per
        for m in range(R):
            for q in range(4):
                want = G["rx"][m * L + r] >> (8 * q) & 255
                assert entry(op, op_words, lane, 4 * m + q) == 8 * (area + want)
        for t in range(G["tot"]):
            code = (G["tc"][t // G["per_word"] * L + r] >> (t % G["per_word"] * G["bits"])
                    & ((1 << G["bits"]) - 1))
            assert entry(tm, tm_words, lane, t) == 8 * (area + G["off_q"] + code)
