"""The schedule autotuner times the kernels that the batch to tune will run: its
samples and cached results stay on their side of the batch sizes at which the
launches change kernels."""
from types import SimpleNamespace

import pytest

from paper_1611_02274_amd import autotune
from paper_1611_02274_amd import codegen as cg
from paper_1611_02274_amd import inputs as I

SIMDS = 1024


def problem(kind, n_sp):
    if kind == "vdp":
        return SimpleNamespace(net=None, kind=kind, n_eq=2)
    if kind == "pleiades":
        return SimpleNamespace(net=None, kind=kind, n_eq=28)
    return SimpleNamespace(net=I.standard_network(n_sp), kind=kind,
                           n_eq=n_sp + (kind == "mass_action_thermal"))


@pytest.mark.parametrize("kind,n_sp,method,n,want", [
    # one lane per system: resident as a whole up to 8 waves of 64 per SIMD
    ("mass_action", 13, "rkc", 300, 300), ("mass_action", 13, "rkc", 1 << 18, 1 << 18),
    ("mass_action_thermal", 9, "rkck", 1 << 20, (1 << 19) + 1), ("vdp", 0, "rkck", 1 << 21,
                                                                 (1 << 19) + 1),
    # one system on several lanes: the wide variants up to so many systems per SIMD
    ("mass_action", 53, "rkck", 1 << 20, 52429), ("mass_action", 53, "rkck", 1 << 17, 16385),
    ("mass_action", 53, "rkck", 16384, 16384), ("mass_action", 32, "rkck", 1 << 18, 49153),
    ("mass_action", 32, "rkck", 40000, 16384), ("mass_action", 32, "rkc", 1 << 18, 16384),
    ("mass_action_thermal", 53, "rkck", 1 << 17, 16384), ("pleiades", 0, "rkck", 1 << 18, 16384)])
def test_sample_runs_the_batch_kernels(kind, n_sp, method, n, want):
    p = problem(kind, n_sp)
    idx = autotune.network_sample(p, method, n, SIMDS, 0.05, 16384, 0)
    assert idx.size == want
    line = autotune.switch_line(p, method, SIMDS)
    assert (idx.size > line) == (n > line)


def test_keys_follow_the_kernels():
    p, th = problem("mass_action", 32), problem("mass_action_thermal", 32)
    key = lambda q, n: autotune.network_key(q, "rkck", n, SIMDS, 1e-8)   # noqa: E731
    assert key(p, 49152) != key(p, 49153) == key(p, 1 << 20)
    assert key(p, 1000) == key(p, 1024) != key(p, 1025)
    assert key(p, 1000) != key(th, 1000)


@pytest.mark.parametrize("n_sp", [32, 53])
def test_limits_are_the_kernels(n_sp):
    net = I.standard_network(n_sp)
    for thermal, text in ((False, cg.wide_source(net, "t")),
                          (True, cg.thermal_group_source(net, "t")[0])):
        for name, method in (("kMaxRkck", "rkck"), ("kMaxRkc", "rkc")):
            assert f"{name} = {cg.wide_limit(n_sp, thermal, method)};" in text
