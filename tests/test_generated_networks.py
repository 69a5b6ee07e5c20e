"""Networks other than the standard four through the code generator: the
sources it writes for them compile for the device (the layouts' static
assertions hold) and their tables name every reaction once."""
import os
import subprocess

import numpy as np
import pytest

from paper_1611_02274_amd import build
from paper_1611_02274_amd import codegen as cg
from paper_1611_02274_amd import inputs as I


def network(n_sp, n_rx, n_third, seed=1):
    """A topology of n_rx reactions between two and two species, n_third of them
    with a one-species side (times [M])."""
    rng = np.random.default_rng(seed)
    reac, prod = np.zeros((n_rx, 2), np.int32), np.zeros((n_rx, 2), np.int32)
    for j in range(n_rx):
        s = rng.choice(n_sp, 4, replace=False)
        reac[j], prod[j] = s[:2], s[2:]
    prod[rng.choice(n_rx, n_third, replace=False), 1] = -1
    z = np.zeros(n_rx)
    return I.Network(n_sp=n_sp, n_rx=n_rx, comp=np.ones((n_sp, 3), np.int64), W=np.ones(n_sp),
                     reac=reac, prod=prod, lnA=z, beta=z, Ea=z, Keq=z + 1.0)


def hipcc(folder, text, *args):
    """Compiles a device source that includes the kernels' headers; its output file."""
    src, out = folder / "net.hip", folder / "net.out"
    src.write_text(text)
    r = subprocess.run([build.HIPCC, *build.CXXFLAGS, "--cuda-device-only", *args,
                        str(src), "-o", str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return out


@pytest.fixture
def folder(tmp_path):
    # the generated headers include the kernels' headers from the folder above
    (tmp_path / "gen").mkdir()
    for f in os.listdir(build.CSRC):
        if f.endswith(".hpp"):
            (tmp_path / f).symlink_to(os.path.join(build.CSRC, f))
    return tmp_path / "gen"


# [M] sides that leave no room for every other reaction in the slots before
# theirs, in the wide layout (all) and in the group layout (the last)
@pytest.mark.parametrize("n_sp,n_rx,n_third", [(17, 49, 16), (32, 96, 16), (53, 365, 92),
                                               (17, 110, 13)])
def test_third_body_slots(folder, n_sp, n_rx, n_third):
    net = network(n_sp, n_rx, n_third)
    for L, G in ((cg.group_lanes(n_sp), cg._group_layout(net, cg.group_lanes(n_sp))),
                 (cg.wide_lanes(n_sp), cg._wide_layout(net, cg.wide_lanes(n_sp)))):
        assert sorted(j for j in G["rx_of"] if j >= 0) == list(range(n_rx))
        third = [p for p, j in enumerate(G["rx_of"])
                 if j >= 0 and (net.reac[j][1] < 0 or net.prod[j][1] < 0)]
        assert G["m_first"] == G["R"] - -(-n_third // L)
        assert min(third) >= G["m_first"] * L
    header, source = cg.rhs_source(net, "t")
    (folder / "net_t.hpp").write_text(header)
    hipcc(folder, source, "-fsyntax-only")


# fewer reaction slots than lanes in [M]'s chain of sums: 53 species in 5 slots
# (seven lanes), 17 in one (three), and one slot more than lanes
@pytest.mark.parametrize("n_sp,n_rx", [(53, 150), (17, 16), (53, 250)])
def test_term_addresses_are_read(folder, n_sp, n_rx):
    """The right-hand side reads the table of its terms' LDS addresses however
    few reaction slots it has (the object holds the table only if it does)."""
    net = network(n_sp, n_rx, 0)
    header, _ = cg.rhs_source(net, "t")
    (folder / "net_t.hpp").write_text(header)
    asm = hipcc(folder, '''#include "net_t.hpp"
using GP = rkmi::gen_t::GNet;
__global__ void rhs(GP::Lane L, double* y) {
  __shared__ __attribute__((aligned(16))) double lds[rkmi::group_lds_doubles<GP>()];
  const rkmi::Grp<GP> x = rkmi::group_of<GP>(lds);
  double a[GP::S], f[GP::S];
  for (int m = 0; m < GP::S; ++m) a[m] = y[m * 64 + threadIdx.x];
  rkmi::group_rhs_mass_action<GP>(L, x, a, f);
  for (int m = 0; m < GP::S; ++m) y[m * 64 + threadIdx.x] = f[m];
}
''', "-S")
    text = asm.read_text()
    assert "kOp" in text and "kTm" in text


# forward RKCK, forward RKC, reverse RKCK, reverse RKC
@pytest.mark.parametrize("n_sp,n_rx,want", [(9, 19, "1111"), (13, 27, "1101"), (12, 40, "0101"),
                                            (16, 50, "0100"), (16, 70, "0000"),
                                            (16, 100, "0000")])
def test_sparse_variant_fits_registers(folder, n_sp, n_rx, want):
    """Small batches take the variant with all rate constants in registers only
    in the kernels that have room for them; the others run the network itself."""
    header, _ = cg.rhs_source(network(n_sp, n_rx, 3), "t")
    (folder / "net_t.hpp").write_text(header)
    asserts = []
    for k, bit in enumerate(want):
        method, reverse = ("kMethodRkck", "kMethodRkc")[k % 2], ("false", "true")[k // 2]
        net = "NetR" if bit == "1" else "Net"
        asserts.append(f"static_assert(std::is_same<Sparse<gen_t::Net, {method}, {reverse}>, "
                       f"gen_t::{net}>::value);")
    hipcc(folder, '#include "net_t.hpp"\nnamespace rkmi {\n' + "\n".join(asserts) + "\n}\n",
          "-fsyntax-only")


@pytest.mark.parametrize("n_sp,n_rx,n_third,shift", [(24, 900, 500, 0), (32, 1000, 600, 3),
                                                     (64, 2100, 1500, 3)])
def test_packed_addresses_of_large_areas(folder, n_sp, n_rx, n_third, shift):
    """Networks whose LDS areas exceed 64 KiB: the packed offsets count doubles,
    and name every operand and term as for smaller ones."""
    net = network(n_sp, n_rx, n_third)
    L = cg.group_lanes(n_sp)
    G = cg._group_layout(net, L)
    assert cg._address_shift(G) == shift
    op, op_words, tm, tm_words = cg._packed_addresses(G)

    def at(table, words, lane, k):   # the double of the workgroup's areas
        byte = (table[lane * words + k // 2] >> (16 * (k % 2)) & 0xffff) << shift
        assert byte % 8 == 0
        return byte // 8

    seen = {j: p for p, j in enumerate(G["rx_of"]) if j >= 0}
    assert len(seen) == n_rx
    terms = cg._species_terms(net)
    for lane in range(64):
        r, area = lane % L, lane // L * G["lds_per_system"]
        for m in range(G["R"]):
            j = G["rx_of"][m * L + r]
            want = [int(k) if k >= 0 else n_sp for k in (*net.reac[j], *net.prod[j])]
            if j >= 0:
                assert [at(op, op_words, lane, 4 * m + q) - area for q in range(4)] == want
        got = [at(tm, tm_words, lane, t) - area - G["off_q"] for t in range(G["tot"])]
        cut = G["bnd"][r] * G["chunk"]
        for part, k in ((got[:cut], G["sp"][r]), (got[cut:], G["sp"][L + r])):
            want = [seen[c >> 1] + G["neg"] * (c & 1) for c in (terms[k] if k >= 0 else [])]
            assert part == want + [G["sentinel"]] * (len(part) - len(want))
    header, source = cg.rhs_source(net, "t")
    (folder / "net_t.hpp").write_text(header)
    hipcc(folder, source, "-fsyntax-only")


@pytest.mark.parametrize("n_sp,kernel", [(13, "ragged_kernel"), (13, "interleaved_kernel"),
                                         (53, "ragged_kernel")])
def test_batches_refuse_the_energy_equation(folder, n_sp, kernel):
    """The batch kernels form no exponentials' table: a batch of a network with
    the energy equation does not compile, the isothermal one does."""
    for thermal in (False, True):
        net = I.thermal_network(n_sp)
        header, _ = (cg.rhs_source(net, "t") if not thermal else cg.thermal_source(net, "t")
                     if n_sp == 13 else cg.thermal_group_source(net, "t"))
        (folder / "net_t.hpp").write_text(header)
        name = "GNet" if thermal and n_sp == 53 else "Net"
        text = (f'#include "net_t.hpp"\n#include "../rk_batch.hpp"\n'
                f"void* f() {{ return (void*)rkmi::{kernel}<rkmi::gen_t::{name}>; }}\n")
        if thermal:
            with pytest.raises(AssertionError, match="cannot enter a ragged batch"):
                hipcc(folder, text, "-fsyntax-only")
        else:
            hipcc(folder, text, "-fsyntax-only")


@pytest.mark.parametrize("n_rx,table", [(302, "true"), (304, "false")])
def test_energy_equation_fits_lds(folder, n_rx, table):
    """One-lane networks with the energy equation whose columns leave no room in
    LDS for the exponentials' table read the constants."""
    header, _ = cg.thermal_source(network(15, n_rx, 3), "t")
    (folder / "net_t.hpp").write_text(header)
    hipcc(folder, '''#include "net_t.hpp"
using namespace rkmi;
using P = gen_t::Net;
static_assert(P::kExpTable == %s);
static_assert(8 * (kernel_lds_doubles<P, kMethodRkc>() * kLdsStride + SharedDoubles<P>::value) <=
              160 << 10);
void* f() { return (void*)plain_kernel<P, kMethodRkc>; }
''' % table, "-fsyntax-only")


def test_small_batches_leave_room(folder):
    """Up to 64 systems per compute unit, a batch of a one-lane network takes at
    most half of the SIMDs (its kernels fill a SIMD's registers), so batches on
    other streams run beside it; every batch is held in waves of 1 to 64 systems."""
    header, source = cg.rhs_source(network(9, 19, 3), "t")
    (folder / "net_t.hpp").write_text(header)
    hipcc(folder, '''#include "net_t.hpp"
#include "../rk_launch.hpp"
using namespace rkmi;
static_assert(WavesPerEu<gen_t::Net>::value > 1, "fills a SIMD");
constexpr bool room(int64_t cus, bool whole_simd) {
  for (int64_t n = 1; n <= 80 * 4 * cus; n += n < 70 * cus ? 1 : 97) {
    const int64_t l = systems_per_wave(n, cus, whole_simd), waves = (n + l - 1) / l;
    if (l < 1 || l > 64 || (waves > 4 * cus && l < 64)) return false;
    if (whole_simd && n <= 64 * cus && waves > 2 * cus) return false;
  }
  return true;
}
static_assert(room(256, true) && room(256, false) && room(64, true));
static_assert(systems_per_wave(4096, 256, false) == 4 && systems_per_wave(4096, 256, true) == 16);
int f(const LaunchArgs* a, hipStream_t s) { return launch_method<gen_t::Net, kMethodRkc, false>(a, s); }
''', "-fsyntax-only", "-fconstexpr-steps=20000000")
