"""Generates the HIP right-hand side of a mass-action network.

The generated code fixes the network's topology (species count and which
species fill each reactant / product slot) at compile time, so every species
index is a constant and the per-system state stays in registers.  Rate
parameters (ln A, b, E, 1/K) and molar masses stay runtime data: they are read
from a uniform device buffer laid out as

    [lnA (n_rx) | beta (n_rx) | Ea (n_rx) | invK (n_rx) | W (n_sp) | invW (n_sp)]

Rate law (Sec. 4.2 species equations with this project's network convention):
C_k = (rho Y_k) / W_k, [M] = sum_k C_k,
q_j = k_f,j prod_R C - k_r,j prod_P C, a one-species side times [M],
k_r,j = k_f,j (1 / K_j), dY_k/dt = (W_k sum_j nu_kj q_j) / rho, with
k_f,j = exp(lnA_j + b_j ln T - E_j / T) formed once per system; divisions by
constants are multiplications by reciprocals formed once.
"""
from __future__ import annotations

import os
import random

import numpy as np

HERE = os.path.dirname(os.path.abspath(__file__))
GEN_DIR = os.path.join(HERE, "csrc", "gen")


def _side(coef, slots):
    a, b = int(slots[0]), int(slots[1])
    second = f"C[{b}]" if b >= 0 else "M"
    return f"({coef} * C[{a}]) * {second}"


# Networks with at most this many species keep their vectors in registers
# (rate constants too); larger ones keep every vector and the rate constants
# in slot columns of the device workspace.
REGISTER_SPECIES_LIMIT = 16
# Larger networks also get a group variant in which several lanes share a
# system: 16 lanes up to 32 species, 32 lanes above.


def group_lanes(n_sp: int) -> int:
    return 16 if n_sp <= 32 else 32


def _gershgorin_source(net) -> str:
    """Gershgorin bound max_k sum_i |J_ki| of the analytic Jacobian at y, in
    the reference evaluation's order: C and [M] as in the right-hand side;
    J_ki = (W_k D_ki) (1/W_i), D_ki the sum over the reactions in order with
    nu_kj != 0 of nu_kj g_ji, g_ji = k_f t_f - k_r t_r, t_f = [r0 = i] X_r1 +
    [r1 = i or empty] C_r0 (t_r likewise); rows summed over i from zero, the
    maximum by fmax from zero.  Entries and terms that are zero by structure
    are left out (adding a zero changes no sum here)."""
    n, nr = net.n_sp, net.n_rx
    lines = ["  static constexpr bool kGershgorin = true;",
             "  template <class VI>",
             "  RKMI_HD static double gershgorin(const Lane& L, const Params& p, const VI& y) {",
             "    const double* __restrict__ iK = p + 3 * NR;",
             "    const double* __restrict__ W = p + 4 * NR;",
             "    const double* __restrict__ iW = W + N;",
             "    const int z = opaque_zero();",
             "    double C[N];",
             "#pragma unroll",
             "    for (int k = 0; k < N; ++k) C[k] = (L.rho * y[k]) * ld_uniform(iW, k);",
             "    double M = 0.0;",
             "#pragma unroll",
             "    for (int k = 0; k < N; ++k) M += C[k];",
             "    double sigma = 0.0;"]

    def x(s):
        return f"C[{s}]" if s >= 0 else "M"
    for k in range(n):
        rx = []
        for j in range(nr):
            r0, r1 = int(net.reac[j][0]), int(net.reac[j][1])
            p0, p1 = int(net.prod[j][0]), int(net.prod[j][1])
            nu = (p0 == k) + (p1 == k) - (r0 == k) - (r1 == k)
            if nu:
                rx.append((j, nu, r0, r1, p0, p1))
        lines.append("    {")
        for j, *_ in rx:
            lines.append(f"      const double kf{j} = L.kf[z + {j} * kLdsStride];")
            lines.append(f"      const double kr{j} = kf{j} * ld_uniform(iK, {j});")
        lines.append("      double r = 0.0;")
        for i in range(n):
            terms = []
            for j, nu, r0, r1, p0, p1 in rx:
                tf = ([x(r1)] if r0 == i else []) + ([x(r0)] if (r1 < 0 or r1 == i) else [])
                tr = ([x(p1)] if p0 == i else []) + ([x(p0)] if (p1 < 0 or p1 == i) else [])
                if not tf and not tr:
                    continue
                fs = f"kf{j} * ({' + '.join(tf)})" if tf else None
                rs = f"kr{j} * ({' + '.join(tr)})" if tr else None
                g = f"{fs} - {rs}" if fs and rs else (fs if fs else f"-({rs})")
                terms.append({1: f"({g})", -1: f"-({g})", 2: f"2.0 * ({g})",
                              -2: f"-2.0 * ({g})"}[nu])
            if terms:
                lines.append(f"      r += fabs((ld_uniform(W, {k}) * ({' + '.join(terms)})) * "
                             f"ld_uniform(iW, {i}));")
        lines.append("      sigma = fmax(sigma, r);")
        lines.append("    }")
    lines += ["    return sigma;", "  }"]
    return "\n".join(lines) + "\n"


def rhs_source(net, tag: str) -> tuple[str, str]:
    """Every operation is written in the order of the reference evaluation
    (products left to right, rate of progress as forward minus reverse, species
    sums accumulated reaction by reaction from zero), and the library is built
    without floating-point contraction, so each rounding is the same."""
    n, nr = net.n_sp, net.n_rx
    columns = n > REGISTER_SPECIES_LIMIT
    lines = []
    for j in range(nr):
        r, p = net.reac[j], net.prod[j]
        lines.append(f"    kf = L.kf[{j} * kLdsStride];" if columns else f"    kf = L.kf[z + {j} * kLdsStride];")
        lines.append(f"    kr = kf * ld_uniform(iK, {j});")
        lines.append(f"    q = {_side('kf', r)} - {_side('kr', p)};")
        for k in r:
            if k >= 0:
                lines.append(f"    om[{int(k)}] -= q;")
        for k in p:
            if k >= 0:
                lines.append(f"    om[{int(k)}] += q;")
    body = "\n".join(lines)
    vjp = "" if columns else _vjp_source(net) + _gershgorin_source(net)
    runs = 0 if columns else sparse_runs(net)
    wide = _sparse_source(net, body, runs) if runs else ""
    group = group_source(net, tag) + wide_source(net, tag) if columns else ""
    fast = (f"template <>\nstruct {'FastVariant' if columns else 'SparseVariant'}<gen_{tag}::Net> "
            f"{{\n  using type = gen_{tag}::{'GNet' if columns else 'NetR'};\n}};\n\n"
            if columns or runs else "")
    if columns:
        launch_call = (f"rkmi::launch_with_wide<rkmi::gen_{tag}::Net, rkmi::gen_{tag}::GNet, "
                       f"rkmi::gen_{tag}::WNet>(a, s)")
        ws_call = (f"rkmi::workspace_with_group<rkmi::gen_{tag}::Net, rkmi::gen_{tag}::GNet>"
                   "(method, schedule, n)")
    else:
        launch_call = f"rkmi::launch<rkmi::gen_{tag}::Net>(a, s)"
        ws_call = f"rkmi::workspace<rkmi::gen_{tag}::Net>(method, schedule, n)"
    if columns:
        storage = """  // vectors and the forward rate constants k_f,j of the system live in slot
  // columns (stride kLdsStride); each k_f,j is read once per evaluation
  static constexpr bool kColumns = true;
  static constexpr int kGroupLanes = 1;
  static constexpr int kLaneDoubles = NR;
  using Params = const double*;
  struct Lane {
    const double* kf;
    double rho, irho;
  };"""
        fill = """    for (int j = 0; j < NR; ++j)
      slot[j * kLdsStride] = crm::cr_exp(p[j] + p[NR + j] * lnT - p[2 * NR + j] / T);
    L.kf = slot;"""
    else:
        storage = """  // vectors live in registers; the forward rate constants k_f,j of the
  // system live in the lane's LDS slot and are read once per evaluation (at an
  // offset the optimizer cannot see through, so the reads and the reverse
  // constants k_f,j / K_j are not hoisted out of the integration loop into
  // ~100 live registers)
  static constexpr bool kColumns = false;
  static constexpr int kGroupLanes = 1;
  static constexpr int kLaneDoubles = NR;
  // two waves per SIMD (the slot, NR + N doubles per lane, fits eight
  // workgroups in a compute unit's LDS up to 13 species and 27 reactions)
  static constexpr int kWavesPerEu = 2;
  using Params = const double*;
  struct Lane {
    const double* kf;
    double rho, irho;
  };"""
        fill = """#pragma nounroll
    for (int j = 0; j < NR; ++j)
      slot[j * kLdsStride] = crm::cr_exp(p[j] + p[NR + j] * lnT - p[2 * NR + j] / T);
    L.kf = slot;"""
    zdecl = "" if columns else "    const int z = opaque_zero();\n"
    header = f"""// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Mass-action network: {n} species, {nr} reversible reactions (topology {tag}).
#pragma once

#include "../rk_adjoint.hpp"
#include "../rk_group.hpp"

namespace rkmi {{
namespace gen_{tag} {{

struct Net {{
  static constexpr int N = {n};
  static constexpr int NR = {nr};
{storage}
  RKMI_HD static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                           int64_t n, double* slot) {{
    const double T = g[i];
    const double rho = g[n + i];
    const double lnT = crm::cr_log(T);
{fill}
    L.rho = rho;
    L.irho = 1.0 / rho;
  }}
  template <class VI, class VO>
  RKMI_HD static void rhs(const Lane& L, const Params& p, const VI& y, VO& f) {{
    const double* __restrict__ iK = p + 3 * NR;
    const double* __restrict__ W = p + 4 * NR;
    const double* __restrict__ iW = W + N;
    double C[N], om[N];
{zdecl}#pragma unroll
    for (int k = 0; k < N; ++k) C[k] = (L.rho * y[k]) * ld_uniform(iW, k);
    double M = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) M += C[k];
#pragma unroll
    for (int k = 0; k < N; ++k) om[k] = 0.0;
    double q, kf, kr;
{body}
#pragma unroll
    for (int k = 0; k < N; ++k) f[k] = (ld_uniform(W, k) * om[k]) * L.irho;
  }}
{vjp}}};
{wide}{group}
}}  // namespace gen_{tag}

{fast}}}  // namespace rkmi
"""
    source = f"""// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Launchers of the {n}-species network (topology {tag}).
#include "net_{tag}.hpp"

extern "C" int rkmi_gen_{tag}_launch(const rkmi::LaunchArgs* a, void* s) {{
  return {launch_call};
}}

extern "C" int rkmi_gen_{tag}_host(const rkmi::LaunchArgs* a) {{
  return rkmi::host_run<rkmi::gen_{tag}::Net>(a);
}}

extern "C" int64_t rkmi_gen_{tag}_workspace(int method, int schedule, int64_t n) {{
  return {ws_call};
}}
{"" if columns else _adjoint_exports(tag)}"""
    return header, source


def _registers(body: str) -> str:
    """A generated evaluation with the rate constants taken from the lane's
    registers."""
    import re
    body = re.sub(r"kf = L\.kf\[z \+ (\d+) \* kLdsStride\];", r"kf = L.kf[\1];", body)
    return re.sub(r"kr = kf \* ld_uniform\(iK, (\d+)\);", r"kr = L.kr[\1];", body)


def sparse_runs(net) -> int:
    """Which kernels of a one-lane network run its sparse variant (rk_device.hpp
    SparseRuns): those whose values fit the 256 doubles of a lane's 512 registers
    beside the rate constants.  Forward RKC: the recursion's vectors, the
    concentrations and the sums, eight doubles per species.  RKCK holds its
    stages at once, eleven per species, and needs room for a stage's products.
    The reverse sweeps add a gradient per reaction.  Times without and with the
    variant at 16000 systems, n species / reactions, ms:
      RKC forward   16/50 23.3, 23.0; 16/60 175, 163; 16/70 97.6, 101
      RKCK forward  12/30 2.61, 2.59; 13/27 1.19, 1.17; 12/40 1.75, 1.89 (8000
                    systems); 16/30 2.53, 3.52; 16/50 1.93, 5.19
      RKC reverse   13/27 20.6, 19.3; 16/30 45.3, 40.2; 15/36 87.8, 82.4; 14/44
                    58.3, 68.3; 16/50 67, 106
      RKCK reverse  9/19 9.74, 8.56; 13/27 (65536 systems) 15.3, 18.6"""
    n, nr = net.n_sp, net.n_rx
    return ((2 * nr + 11 * n <= 200) | (2 * nr + 8 * n <= 256) << 1 |
            (3 * nr + 6 * n <= 128) << 2 | (3 * nr + 6 * n <= 200) << 3)


def _sparse_source(net, body: str, runs: int) -> str:
    """The network with both rate constants of every reaction in registers,
    compiled for one wave per SIMD: batches that do not put a second wave on a
    SIMD (rk_device.hpp SparseVariant)."""
    return f"""
// The same network for batches of at most one wave per SIMD: such a wave has
// the SIMD's registers to itself and nothing to hide latency behind, so both
// rate constants of every reaction stay in registers (no LDS read of k_f, no
// scalar load of 1/K, no k_r product per evaluation).  9 species RKC, 300 systems
// 21.5 -> 16.4 ms, RKCK 5001 13.4 -> 10.2 ms; 13 species RKC 65536 systems 13.8 ->
// 12.1 ms, its reverse sweep 2^16 systems 23.3 -> 22.2 ms; 9 species RKCK forward
// and back, 65536 systems, 91.9 -> 84.7 ms.
struct NetR {{
  static constexpr int N = Net::N;
  static constexpr int NR = Net::NR;
  static constexpr bool kColumns = false;
  static constexpr int kGroupLanes = 1;
  static constexpr int kLaneDoubles = NR;   // set-up only
  static constexpr int kWavesPerEu = 1;
  // kernels whose registers it fits (forward RKCK, RKC, then the reverse sweeps)
  static constexpr int kRuns = {runs};
  using Params = Net::Params;
  struct Lane {{
    double kf[NR], kr[NR];
    double rho, irho;
  }};
  RKMI_HD static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                           int64_t n, double* slot) {{
    Net::Lane s;
    Net::init(s, p, g, i, n, slot);
#pragma unroll
    for (int j = 0; j < NR; ++j) {{
      L.kf[j] = slot[j * kLdsStride];
      L.kr[j] = L.kf[j] * ld_uniform(p, 3 * NR + j);
    }}
    L.rho = s.rho;
    L.irho = s.irho;
  }}
  template <class VI, class VO>
  RKMI_HD static void rhs(const Lane& L, const Params& p, const VI& y, VO& f) {{
    const double* __restrict__ W = p + 4 * NR;
    const double* __restrict__ iW = W + N;
    double C[N], om[N];
#pragma unroll
    for (int k = 0; k < N; ++k) C[k] = (L.rho * y[k]) * ld_uniform(iW, k);
    double M = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) M += C[k];
#pragma unroll
    for (int k = 0; k < N; ++k) om[k] = 0.0;
    double q, kf, kr;
{_registers(body)}
#pragma unroll
    for (int k = 0; k < N; ++k) f[k] = (ld_uniform(W, k) * om[k]) * L.irho;
  }}
{_registers(_vjp_source(net))}}};
"""


def thermal_source(net, tag: str) -> tuple[str, str]:
    """The network with the energy equation (Sec. 4.2 at constant volume):
    state (T, Y_1..Y_N), one parameter per system (rho); the rate coefficients
    are evaluated at the current T in every evaluation (a rolled loop through
    the lane's LDS slot, one copy of the exponential's code), the species part
    is the isothermal rate law, and dT/dt = -((sum_k (e_k omega_k) W_k / rho) /
    c_v).  Same operations in the same order as the reference evaluation.
    Systems of up to 16 unknowns keep their vectors in registers."""
    n, nr = net.n_sp, net.n_rx
    assert n + 1 <= REGISTER_SPECIES_LIMIT
    # exponentials side by side: the divisor of the reactions, rounded up, in 3..5
    # that wastes least
    K = min((3, 4, 5), key=lambda k: (-nr % k, k))
    # their tables in LDS beside the lanes' columns, unless these fill its 160 KiB
    table = 64 * 8 * (nr + n + 1) + 8 * 128 <= 160 << 10
    lines = []
    for j in range(nr):
        r, p = net.reac[j], net.prod[j]
        lines.append(f"    kf = L.kf[z + {j} * kLdsStride];")
        lines.append(f"    kr = kf * ld_uniform(iK, {j});")
        lines.append(f"    q = {_side('kf', r)} - {_side('kr', p)};")
        for k in r:
            if k >= 0:
                lines.append(f"    om[{int(k)}] -= q;")
        for k in p:
            if k >= 0:
                lines.append(f"    om[{int(k)}] += q;")
    body = "\n".join(lines)
    header = f"""// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Mass-action network with the energy equation: {n} species + T, {nr} reversible
// reactions (topology {tag}).
#pragma once

#include "../rk_launch.hpp"

namespace rkmi {{
namespace gen_{tag} {{

struct Net {{
  static constexpr int NS = {n};
  static constexpr int N = NS + 1;
  static constexpr int NR = {nr};
  // vectors in registers; k_f,j(T) of the current evaluation in the lane's LDS
  // slot, read back at an offset the optimizer cannot see through
  static constexpr bool kColumns = false;
  static constexpr int kGroupLanes = 1;
  static constexpr int kLaneDoubles = NR;
  static constexpr int kWavesPerEu = 2;
  static constexpr bool kExpTable = {str(table).lower()};
  // uniform data: [lnA | beta | Ea | 1/K | W | 1/W | u0 | cv0 | cv1]
  using Params = const double*;
  struct Lane {{
    double* kf;
{"    crm::ExpTable et;" if table else "    crm::ExpConstants et;"}
    double rho, irho;
  }};
  RKMI_HD static void init(Lane& L, const Params&, const double* __restrict__ g, int64_t i,
                           int64_t, double* slot) {{
    L.kf = slot;
{"    L.et.p = shared_area<Net>(slot);" if table else ""}
    L.rho = g[i];
    L.irho = 1.0 / L.rho;
  }}
  template <class VI, class VO>
  RKMI_HD static void rhs(const Lane& L, const Params& p, const VI& y, VO& f) {{
    // (constants at an offset the optimizer cannot see through: hoisted out of the
    // integration loop they overflow the scalar registers, and reading them back
    // from vector lanes cost 3 %)
    const int z = opaque_zero();
    const double* __restrict__ iK = p + 3 * NR + z;
    const double* __restrict__ W = p + 4 * NR + z;
    const double* __restrict__ iW = W + NS;
    const double* __restrict__ u0 = W + 2 * NS;
    const double* __restrict__ cv0 = W + 3 * NS;
    const double* __restrict__ cv1 = W + 4 * NS;
    const double T = y[0];
    const double lnT = crm::cr_log(T);
    const double invT = 1.0 / T;
    // {K} exponentials side by side without a branch, their tables in LDS: one at a
    // time, each waited out its table reads and its own chain of operations (9
    // species 65536 systems 178 -> 114 ms, 13 species 84 -> 54 ms)
#pragma nounroll
    for (int j0 = 0; j0 < NR; j0 += {K}) {{
      double a[{K}], e[{K}];
#pragma unroll
      for (int k = 0; k < {K}; ++k) {{
        const int j = j0 + k < NR ? j0 + k : NR - 1;
        a[k] = ld_uniform(p, j) + ld_uniform(p, NR + j) * lnT - ld_uniform(p, 2 * NR + j) * invT;
      }}
      crm::cr_exp_n<{K}>(a, e, L.et);
#pragma unroll
      for (int k = 0; k < {K}; ++k)
        L.kf[z + (j0 + k < NR ? j0 + k : NR - 1) * kLdsStride] = e[k];
    }}
    double C[NS], om[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) C[k] = (L.rho * y[1 + k]) * ld_uniform(iW, k);
    double M = 0.0;
#pragma unroll
    for (int k = 0; k < NS; ++k) M += C[k];
#pragma unroll
    for (int k = 0; k < NS; ++k) om[k] = 0.0;
    double q, kf, kr;
{body}
#pragma unroll
    for (int k = 0; k < NS; ++k) f[1 + k] = (ld_uniform(W, k) * om[k]) * L.irho;
    double sum = 0.0, cv = 0.0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {{
      const double e = ld_uniform(u0, k) + (ld_uniform(cv0, k) + ld_uniform(cv1, k) * T) * T;
      sum += (e * om[k]) * ld_uniform(W, k);
      cv += y[1 + k] * (ld_uniform(cv0, k) + 2.0 * ld_uniform(cv1, k) * T);
    }}
    f[0] = -((sum * L.irho) / cv);
  }}
}};

// Batches of at most one wave per SIMD: the wave has the SIMD's registers to
// itself.
struct NetR : Net {{
  static constexpr int kWavesPerEu = 1;
}};

}}  // namespace gen_{tag}

template <>
struct SparseVariant<gen_{tag}::Net> {{
  using type = gen_{tag}::NetR;
}};

}}  // namespace rkmi
"""
    source = f"""// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Launchers of the {n}-species network with the energy equation (topology {tag}).
#include "net_{tag}.hpp"

extern "C" int rkmi_gen_{tag}_launch(const rkmi::LaunchArgs* a, void* s) {{
  return rkmi::launch<rkmi::gen_{tag}::Net>(a, s);
}}

extern "C" int rkmi_gen_{tag}_host(const rkmi::LaunchArgs* a) {{
  return rkmi::host_run<rkmi::gen_{tag}::Net>(a);
}}

extern "C" int64_t rkmi_gen_{tag}_workspace(int method, int schedule, int64_t n) {{
  return rkmi::workspace<rkmi::gen_{tag}::Net>(method, schedule, n);
}}
"""
    return header, source


def thermal_group_source(net, tag: str) -> tuple[str, str]:
    """The network with the energy equation on the group schedule (32 lanes per
    system, rk_group.hpp group_rhs_thermal) and, for small batches, one unknown
    per lane of a wave (group_rhs_thermal_wide): unknowns (T, Y_1..Y_N), the
    rate coefficients k_f,j(T) formed by each position's lane at every
    evaluation, and dT/dt from two species sums.  Same operations in the same
    order as the reference evaluation."""
    n, nr = net.n_sp, net.n_rx
    G = _group_layout(net, 32, thermal=True)
    W = _wide_layout(net, 64, thermal=True)
    kg, kw = (min((3, 4, 5), key=lambda k: (-X["R"] % k, k)) for X in (G, W))
    prm = 4 * nr + 5 * n + (4 * nr + 5 * n) % 2
    header = f"""// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Mass-action network with the energy equation on the group schedule: {n} species
// + T, {nr} reversible reactions (topology {tag}).
#pragma once

#include "../rk_launch.hpp"
#include "../rk_group.hpp"

namespace rkmi {{
namespace gen_{tag} {{

struct GNet {{
  static constexpr bool kThermal = true;
  static constexpr bool kExpTable = true;
  static constexpr int NS = {n};
  static constexpr int N = NS + 1;    // unknowns: T, then the species
  static constexpr int NR = {nr};
  static constexpr int kL = {G["L"]};
  static constexpr int kGroupLanes = {G["L"]};
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  static constexpr int kWavesPerEuRkc = 2;
  static constexpr int kWavesPerEuRkck = 2;
  static constexpr int S = {G["S"]};
  static constexpr int R = {G["R"]};
  static constexpr int kExps = {kg};    // exponentials formed side by side
  static constexpr int kMSlot = {G["m_first"]};   // first slot that may hold a [M] reaction
  static constexpr int kOffC = 0;
  static constexpr int kOffT = NS + 1;            // T, written by its owner
  static constexpr int kOffQ = {G["off_q"]};
  static constexpr int kSentinel = {G["sentinel"]};
  static constexpr int kNegOff = {G["neg"]};
  static constexpr int kOffRed = {G["off_red"]};
  static constexpr int kOffE1 = {G["off_e1"]};   // the energy sum's terms (after the RKC coefficients)
  static constexpr int kOffE2 = {G["off_e2"]};   // the heat capacity's terms
  static constexpr int kLdsPerSystem = {G["lds_per_system"]};
  static constexpr int kTermLen = {G["tot"]};
  static constexpr int kChunk = {G["chunk"]};
  // uniform data: [lnA | beta | Ea | 1/K | W | 1/W | u0 | cv0 | cv1], then (lnA,
  // beta, Ea, 1/K) of each position's reaction, here and in the wide variant
  static constexpr int kPrmOffset = {prm};
  using Params = const double*;
{_group_tables(G)}
  struct Lane {{
    const double* prm;   // the uniform data (rate parameters read at every evaluation)
    crm::ExpTable et;
    double W[S], iW[S], u0[S], cv0[S], cv1[S];
    double rho, irho;
    int bnd;   // chunks of the slot-0 list
  }};
  __device__ static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                              int64_t, const Grp<GNet>& x) {{
    L.prm = p;
    L.et = shared_exp_table(x);
#pragma unroll
    for (int m = 0; m < S; ++m) {{
      const int k = x.sp[m] - 1;   // species of the slot (T and empty slots: none)
      const bool sp = k >= 0;
      L.W[m] = sp ? p[4 * NR + k] : 0.0;
      L.iW[m] = sp ? p[4 * NR + NS + k] : 0.0;
      L.u0[m] = sp ? p[4 * NR + 2 * NS + k] : 0.0;
      L.cv0[m] = sp ? p[4 * NR + 3 * NS + k] : 0.0;
      L.cv1[m] = sp ? p[4 * NR + 4 * NS + k] : 0.0;
    }}
    L.rho = g[i];
    L.irho = 1.0 / L.rho;
    L.bnd = kBnd[x.r];
    // the zero that pads the term sequences
    if (x.r == 0) x.lds[kOffQ + kSentinel] = 0.0;
  }}
}};

// Wide variant: one unknown per lane of a wave (rk_group.hpp).
struct WNet {{
  static constexpr bool kThermal = true;
  static constexpr bool kWide = true;
  // largest batches it runs, in systems per SIMD (rk_group.hpp group_rhs_thermal_wide)
  static constexpr int kMaxRkck = {wide_limit(n, True, 'rkck')};
  static constexpr int kMaxRkc = {wide_limit(n, True, 'rkc')};
  static constexpr bool kExpTable = true;
  static constexpr int NS = {n};
  static constexpr int N = NS + 1;    // unknowns: T, then the species
  static constexpr int NR = {nr};
  static constexpr int kL = 64;
  static constexpr int kGroupLanes = 64;
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  static constexpr int kWavesPerEuRkc = 1;
  static constexpr int kWavesPerEuRkck = 1;
  static constexpr int S = 1;
  static constexpr int R = {W["R"]};
  static constexpr int kExps = {kw};    // exponentials formed side by side
  static constexpr int kMSlot = {W["m_first"]};   // first slot that may hold a [M] reaction
  static constexpr int kOffC = 0;
  static constexpr int kOffQ = {W["off_q"]};
  static constexpr int kOffZero = {W["off_zero"]};
  static constexpr int kNegOff = {W["neg"]};
  static constexpr int kOffRed = {W["off_red"]};
  static constexpr int kOffE1 = {W["off_e1"]};   // the energy sum's terms (after the RKC coefficients)
  static constexpr int kOffE2 = {W["off_e2"]};   // the heat capacity's terms
  static constexpr int kLdsPerSystem = {W["lds"]};
  static constexpr int kTermLen = {W["T"]};
  static constexpr int kPrmOffset = GNet::kPrmOffset + 4 * GNet::R * GNet::kL;
  using Params = const double*;
{_table("kSp", "int", [r if r <= n else -1 for r in range(64)])}
{_table("kRxOf", "int16_t", W["rx_of"])}
  // LDS byte offsets within the system's area: each lane's rate operands
  // (R x 4), and the signed rates of its species in reaction order
{_table("kOp", "uint16_t", W["ops"], align=16)}
{_table("kTm", "uint16_t", W["tm"], align=16)}
  struct Lane {{
    const double* prm;   // the uniform data (rate parameters read at every evaluation)
    crm::ExpTable et;
    double W[S], iW[S], u0[S], cv0[S], cv1[S];
    double rho, irho;
    uint32_t op[R][4], tm[kTermLen];   // LDS addresses, formed once per system
    uint32_t c_at;
  }};
  __device__ static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                              int64_t, const Grp<WNet>& x) {{
    L.prm = p;
    L.et = shared_exp_table(x);
    const int k = x.sp[0] - 1;   // species of the lane (T and empty lanes: none)
    const bool sp = k >= 0;
    L.W[0] = sp ? p[4 * NR + k] : 0.0;
    L.iW[0] = sp ? p[4 * NR + NS + k] : 0.0;
    L.u0[0] = sp ? p[4 * NR + 2 * NS + k] : 0.0;
    L.cv0[0] = sp ? p[4 * NR + 3 * NS + k] : 0.0;
    L.cv1[0] = sp ? p[4 * NR + 4 * NS + k] : 0.0;
    L.rho = g[i];
    L.irho = 1.0 / L.rho;
    const uint32_t base = lds_address(x.lds);
    L.c_at = base + 8 * (sp ? k : NS + 1);
#pragma unroll
    for (int q = 0; q < 4 * R; ++q) L.op[q / 4][q % 4] = base + kOp[x.r * 4 * R + q];
#pragma unroll
    for (int t = 0; t < kTermLen; ++t) L.tm[t] = base + kTm[x.r * kTermLen + t];
    if (x.r == 0) x.lds[kOffZero] = 0.0;
  }}
}};

}}  // namespace gen_{tag}
}}  // namespace rkmi
"""
    source = f"""// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Launchers of the {n}-species network with the energy equation (topology {tag}): the
// group kernels under every schedule; no host build of the per-system code.
#include "net_{tag}.hpp"

extern "C" int rkmi_gen_{tag}_launch(const rkmi::LaunchArgs* a, void* s) {{
  return rkmi::launch_group_only<rkmi::gen_{tag}::GNet, rkmi::gen_{tag}::WNet>(a, s);
}}

extern "C" int rkmi_gen_{tag}_host(const rkmi::LaunchArgs*) {{
  return rkmi::kLaunchInvalid;
}}

extern "C" int64_t rkmi_gen_{tag}_workspace(int, int, int64_t n) {{
  return n > 0 ? (int64_t)rkmi::kQueueBytes : 0;
}}

namespace rkmi {{
RateOrder gen_{tag}_rates(int k) {{
  using G = gen_{tag}::GNet;
  using W = gen_{tag}::WNet;
  return k == 0 ? RateOrder{{G::kRxOf, G::R * G::kL, G::kPrmOffset}}
                : RateOrder{{W::kRxOf, W::R * W::kL, W::kPrmOffset}};
}}
}}  // namespace rkmi
"""
    return header, source


def _species_terms(net):
    """Per species, the signed rates of its omega sum in evaluation order:
    reaction by reaction, reactant slots (subtract) before product slots (add).
    Entries are q_index << 1 | negative."""
    terms = [[] for _ in range(net.n_sp)]
    for j in range(net.n_rx):
        for k in net.reac[j]:
            if k >= 0:
                terms[int(k)].append(j << 1 | 1)
        for k in net.prod[j]:
            if k >= 0:
                terms[int(k)].append(j << 1)
    return terms


def _table(name, ctype, values, per_line=16, align=0):
    rows = [", ".join(str(v) for v in values[i:i + per_line])
            for i in range(0, len(values), per_line)]
    body = ",\n      ".join(rows)
    al = f"alignas({align}) " if align else ""
    return f"  {al}static constexpr {ctype} {name}[{len(values)}] = {{\n      {body}}};"


# Group variants: a lane's species list is consumed in chunks of this many
# terms; its first species' list is padded to a whole number of chunks.
GROUP_TERM_CHUNK = 4
# doubles of the group scratch that hold the RKC stage recurrence (RkcCoef, 11
# doubles) between evaluations for stage counts above the tabulated ones
GROUP_COEF_DOUBLES = 12


def _group_positions(net, L, R):
    """Reaction -> rate position p = m * L + r (slot m of lane r).  Reactions
    with a one-species side (times [M]) fill the last slots, so the kernel
    selects [M] for an operand only there; the others fill the first slots in
    reaction order.  Returns (position of each reaction, reaction of each
    position or -1, first slot that may hold a [M] reaction)."""
    nr, n = net.n_rx, net.n_sp
    third = [j for j in range(nr) if int(net.reac[j][1]) < 0 or int(net.prod[j][1]) < 0]
    plain = [j for j in range(nr) if j not in set(third)]
    m_slots = -(-len(third) // L) if third else 0
    # the [M] slots also take the plain reactions that do not fit before them
    # (R slots hold all reactions, so what is left of these fits there)
    m_first = R - m_slots
    front = plain[:m_first * L]
    back = plain[m_first * L:] + third
    assert len(back) <= (R - m_first) * L
    pos_of = [-1] * nr
    rx_of = [-1] * (R * L)
    for p, j in enumerate(front):
        pos_of[j], rx_of[p] = p, j
    for t, j in enumerate(back):
        p = m_first * L + t
        pos_of[j], rx_of[p] = p, j
    return pos_of, rx_of, (m_first if third else R)


def _spread_banks(net, L, R, m_first, pos_of, rx_of, seqs, neg, off_q, zero, area):
    """Rearranges the reactions over their positions, within the slots before
    m_first and those from it on, so that a wave's reads of LDS meet in fewer
    banks: a 64-lane read of doubles takes the sum over its two halves of the
    most addresses in one of the 32 banks (measured: 3.1 cycles at one each, 4.6
    at two, 8.5 at four).  seqs[r] is the sequence of lane r's terms ((reaction,
    1 if negative) or None, the zero at `zero`), area the doubles of a system; a
    deterministic local search."""
    rng = random.Random(1)
    steps = max(len(q) for q in seqs)
    reads = steps + 4 * R           # the terms' reads, then the operands'
    refs = [({}, {}) for _ in range(reads)]
    load = [([0] * 32, [0] * 32) for _ in range(reads)]
    lanes = [[((g * L + r) // 32, g * area) for g in range(64 // L)] for r in range(L)]
    species = [[int(k) if k >= 0 else net.n_sp for k in (*net.reac[j], *net.prod[j])]
               for j in range(net.n_rx)]
    uses = [[] for _ in range(net.n_rx)]

    def count(i, r, a, d):
        for h, off in lanes[r]:
            c = refs[i][h].get(a + off, 0) + d
            refs[i][h][a + off] = c
            if c == max(d, 0):      # the address came or went
                load[i][h][(a + off) % 32] += d

    def place(j, p, d):
        r, m = p % L, p // L
        for q in range(4):
            count(steps + 4 * m + q, r, species[j][q] if j >= 0 else 0, d)
        for t, rr, minus in uses[j] if j >= 0 else ():
            count(t, rr, off_q + p + neg * minus, d)

    def cost(i):
        return max(load[i][0]) + max(load[i][1])

    for r in range(L):
        for t, e in enumerate(seqs[r]):
            if e is None:
                count(t, r, zero, 1)
            else:
                uses[e[0]].append((t, r, e[1]))
    for p, j in enumerate(rx_of):
        place(j, p, 1)
    costs = [cost(i) for i in range(reads)]
    for _ in range(12000):
        a = rng.randrange(R * L)
        b = rng.randrange(m_first * L) if a < m_first * L else rng.randrange(m_first * L, R * L)
        ja, jb = rx_of[a], rx_of[b]
        if ja == jb:
            continue
        place(ja, a, -1), place(jb, b, -1), place(ja, b, 1), place(jb, a, 1)
        touched = {t for j in (ja, jb) if j >= 0 for t, _, _ in uses[j]}
        touched |= {steps + 4 * (p // L) + q for p in (a, b) for q in range(4)}
        after = {i: cost(i) for i in touched}
        if sum(after.values()) > sum(costs[i] for i in touched):
            place(ja, b, -1), place(jb, a, -1), place(ja, a, 1), place(jb, b, 1)
            continue
        for i, c in after.items():
            costs[i] = c
        for j, p in ((ja, b), (jb, a)):
            rx_of[p] = j
            if j >= 0:
                pos_of[j] = p


def _group_species(lens, L, chunk):
    """Species -> (lane, slot) for two slots per lane: each lane sums its
    slot-0 species' terms (padded to whole chunks), then its slot-1 species'.
    The heaviest lists go alone to a lane (in slot 1: no padding); the rest
    are paired heavy with light, each pair ordered for the shorter padded
    sequence.  Returns sp[slot * L + lane] (-1: none)."""
    n = len(lens)
    assert L < n <= 2 * L
    order = sorted(range(n), key=lambda k: (-lens[k], k))
    single = 2 * L - n
    sp = [-1] * (2 * L)
    for r in range(single):
        sp[L + r] = order[r]
    rest = order[single:]
    m = len(rest)

    def padded(k):
        return -(-lens[k] // chunk) * chunk

    for i in range(m // 2):
        a, b = rest[i], rest[m - 1 - i]
        if padded(b) + lens[a] < padded(a) + lens[b]:
            a, b = b, a
        sp[single + i] = a
        sp[L + single + i] = b
    return sp


def _group_layout(net, L, thermal=False):
    """The group layout of a network (rk_group.hpp): reaction positions,
    operand codes, the unknowns of each lane's slots (isothermal: species k
    is unknown k; with the energy equation T is unknown 0 and species k is
    unknown 1 + k), the LDS area and each lane's packed term sequence."""
    n, nr = net.n_sp, net.n_rx
    nu = n + 1 if thermal else n          # unknowns
    S, R = -(-nu // L), -(-nr // L)
    assert S == 2, "group variants hold two unknowns per lane"
    assert n < 255, "species indices are packed in bytes"
    chunk = GROUP_TERM_CHUNK
    pos_of, rx_of, m_first = _group_positions(net, L, R)
    # LDS area of a system (doubles): C [0, NS] (C_N the [M] operand's place;
    # with the energy equation T at NS + 1) | rates +q at kOffQ + p, p < R*L,
    # the zero at kOffQ + R*L, scratch (16-byte aligned: the norms over the
    # unknowns; with the energy equation also two species sums) | -q at
    # kOffQ + kNegOff + p
    c_len = n + (2 if thermal else 1)
    off_q = c_len + c_len % 2
    off_red = off_q + R * L + 1 + (off_q + R * L + 1) % 2
    # with the energy equation the two species rows follow the RKC recurrence's
    # coefficients, which stay in the scratch across evaluations
    off_e1 = off_red + GROUP_COEF_DOUBLES
    off_e2 = off_e1 + n + n % 2
    red_len = max(nu, off_e2 + n + n % 2 - off_red) if thermal else nu
    neg = off_red - off_q + red_len
    lds_per_system = off_q + neg + R * L
    lds_per_system += lds_per_system % 2
    sentinel = R * L
    sterms = [[(c >> 1, c & 1) for c in lst] for lst in _species_terms(net)]
    terms = ([[]] + sterms) if thermal else sterms     # per unknown
    lens = [len(t) for t in terms]
    sp = _group_species(lens, L, chunk)
    seqs, bnd = [], []
    for r in range(L):
        k0, k1 = sp[r], sp[L + r]
        l0 = terms[k0] if k0 >= 0 else []
        l0 = l0 + [None] * ((-len(l0)) % chunk)
        l1 = terms[k1] if k1 >= 0 else []
        seqs.append(l0 + l1)
        bnd.append(len(l0) // chunk)
    tot = max(len(q) for q in seqs)
    tot += (-tot) % chunk
    assert tot // chunk <= 64
    seqs = [q + [None] * (tot - len(q)) for q in seqs]
    _spread_banks(net, L, R, m_first, pos_of, rx_of, seqs, neg, off_q, off_q + sentinel,
                  lds_per_system)
    seqs = [[sentinel if e is None else pos_of[e[0]] + neg * e[1] for e in q] for q in seqs]
    rx = []
    for p in range(R * L):
        j = rx_of[p]
        if j >= 0:
            a, b = int(net.reac[j][0]), int(net.reac[j][1])
            c, d = int(net.prod[j][0]), int(net.prod[j][1])
            b = n if b < 0 else b
            d = n if d < 0 else d
            rx.append(a | b << 8 | c << 16 | d << 24)
        else:
            rx.append(0)
    bits = (neg + R * L).bit_length()
    per_word = 32 // bits
    n_words = max(1, -(-tot // per_word))
    tc = [0] * (n_words * L)
    for r in range(L):
        for t, code in enumerate(seqs[r]):
            tc[(t // per_word) * L + r] |= code << ((t % per_word) * bits)
    return dict(n=n, nr=nr, nu=nu, L=L, S=S, R=R, m_first=m_first, rx=rx, rx_of=rx_of,
                off_q=off_q, off_red=off_red, off_e1=off_e1, off_e2=off_e2, neg=neg,
                lds_per_system=lds_per_system,
                sentinel=sentinel, sp=sp, bnd=bnd, tot=tot, bits=bits, per_word=per_word,
                n_words=n_words, tc=tc, chunk=chunk,
                switch=sum(1 << (b - 1) for b in set(bnd) if b > 0))


def _group_tables(G) -> str:
    op, op_words, tm, tm_words = _packed_addresses(G)
    return f"""{_table("kSp", "int", G["sp"])}
{_table("kRxOf", "int16_t", G["rx_of"])}
  // each lane's LDS offsets (in units of 2^kAddrShift bytes) in the wave's areas,
  // two to a word, contiguous and 16-byte aligned (read as whole vectors at every
  // evaluation): the rates' operands, the terms
  static constexpr int kAddrShift = {_address_shift(G)};
  static constexpr int kOpWords = {op_words};
  static constexpr int kTmWords = {tm_words};
{_table("kOp", "uint32_t", op, align=16)}
{_table("kTm", "uint32_t", tm, align=16)}
{_table("kBnd", "int", G["bnd"])}
  // chunks at whose end some lane moves its accumulator to slot 0 (bit c)
  static constexpr uint64_t kSwitchChunks = {G["switch"]}ull;"""


def _address_shift(G) -> int:
    """Unit of the packed LDS offsets: bytes, or doubles for areas beyond 64 KiB
    (networks of about a thousand reactions), whose reads then cost a shift."""
    return 0 if 8 * (64 // G["L"]) * G["lds_per_system"] <= 1 << 16 else 3


def _packed_addresses(G):
    """Offsets in a wave's LDS areas (_address_shift), two to a word, each lane's
    words contiguous and padded to whole 16-byte vectors: its rate operands (four
    per slot) and the terms of its species' sums, from the layout's codes.
    Returns (operand words, words per lane, term words, words per lane)."""
    L, R, bits, per_word = G["L"], G["R"], G["bits"], G["per_word"]
    unit = 8 >> _address_shift(G)

    def packed(entry, count):
        out = []
        for lane in range(64):
            v = [unit * (entry(k, lane % L) + lane // L * G["lds_per_system"])
                 for k in range(count)]
            assert max(v) < 1 << 16
            v += [0] * (-count % 8)
            out += [a | b << 16 for a, b in zip(v[::2], v[1::2])]
        return out, len(out) // 64

    return (*packed(lambda k, r: G["rx"][k // 4 * L + r] >> (8 * (k % 4)) & 255, 4 * R),
            *packed(lambda k, r: G["off_q"] + (G["tc"][k // per_word * L + r]
                                               >> (k % per_word * bits) & ((1 << bits) - 1)),
                    G["tot"]))


def group_source(net, tag: str, lanes: int | None = None) -> str:
    """The group variant of a network (kernels of rk_group.hpp): lane r of a
    group of `lanes` computes the rates of progress at its positions
    p = m*lanes + r (_group_positions) and owns the species of its two slots
    (_group_species); per lane: the species of each slot, the LDS offsets of
    each position's operands and those of its species' signed rates in reaction
    order (slot 0's list, padded to whole chunks, then slot 1's)."""
    n, nr = net.n_sp, net.n_rx
    L = lanes or group_lanes(n)
    G = _group_layout(net, L)
    S, R, m_first = G["S"], G["R"], G["m_first"]
    off_q, sentinel, neg, off_red = G["off_q"], G["sentinel"], G["neg"], G["off_red"]
    lds_per_system = G["lds_per_system"]
    tot, chunk = G["tot"], G["chunk"]
    return f"""
// Group variant: {L} lanes per system (rk_group.hpp).
struct GNet {{
  static constexpr int N = {n};
  static constexpr int NR = {nr};
  static constexpr int kL = {L};
  static constexpr int kGroupLanes = {L};
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  // RKCK: three waves per SIMD, its loop fits 168 registers but for a few spills
  // outside the evaluations (53 species, 65536 systems, in one session: three waves
  // 636 ms, two 698)
  static constexpr int kWavesPerEuRkc = 2;
  static constexpr int kWavesPerEuRkck = 3;
  static constexpr int S = {S};
  static constexpr int R = {R};
  static constexpr int kMSlot = {m_first};   // first slot that may hold a [M] reaction
  static constexpr int kOffC = 0;
  static constexpr int kOffQ = {off_q};
  static constexpr int kSentinel = {sentinel};
  static constexpr int kNegOff = {neg};
  static constexpr int kOffRed = {off_red};
  static constexpr int kLdsPerSystem = {lds_per_system};
  static constexpr int kTermLen = {tot};
  static constexpr int kChunk = {chunk};
  using Params = const double*;
{_group_tables(G)}
  struct Lane {{
    double kf[R], kr[R];
    double W[S], iW[S];
    double rho, irho;
    int bnd;   // chunks of the slot-0 list
  }};
  // The forward rate constants of a lane's positions into the group's rate
  // area; once per system, out of line (the exponentials' temporaries do not
  // count against the registers of the evaluation loop).
  __device__ __attribute__((noinline)) static void rates(Params p, double T, double* lds, int r) {{
    const double lnT = crm::cr_log(T);
    double* const Q = lds + kOffQ;
#pragma nounroll
    for (int m = 0; m < R; ++m) {{
      const int j = kRxOf[m * kL + r];
      if (j >= 0) Q[m * kL + r] = crm::cr_exp(p[j] + p[NR + j] * lnT - p[2 * NR + j] / T);
    }}
  }}
  __device__ static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                              int64_t n, const Grp<GNet>& x) {{
    const double T = g[i];
    const double rho = g[n + i];
    double* const Q = x.lds + kOffQ;
    rates(p, T, x.lds, x.r);
#pragma unroll
    for (int m = 0; m < R; ++m) {{
      const int j = kRxOf[m * kL + x.r];
      L.kf[m] = j >= 0 ? Q[m * kL + x.r] : 0.0;
      L.kr[m] = j >= 0 ? L.kf[m] * p[3 * NR + j] : 0.0;
    }}
#pragma unroll
    for (int m = 0; m < S; ++m) {{
      const int k = x.sp[m];
      L.W[m] = k >= 0 ? p[4 * NR + k] : 0.0;
      L.iW[m] = k >= 0 ? p[4 * NR + N + k] : 0.0;
    }}
    L.rho = rho;
    L.irho = 1.0 / rho;
    L.bnd = kBnd[x.r];
    if (x.r == 0) Q[kSentinel] = 0.0;
  }}
}};
"""


def wide_limit(n_sp: int, thermal: bool, method: str) -> int:
    """Systems per SIMD up to which a network's wide variant runs a batch: measured
    on the 32- and 53-species networks (rk_group.hpp group_rhs_wide,
    group_rhs_thermal_wide).  Seven networks of 17 to 60 species and 60 to 300
    reactions, against the group kernels before the variant came: 1.04 to 2.8 times
    faster up to these lines, but for 20 and 26 species RKCK at 48000 systems (0.94
    and 0.97 times) and 60 species + T RKCK at 12000 (0.99)."""
    if thermal:
        return 1 if method == "rkc" else 6 if n_sp <= 32 else 12
    return (6 if n_sp <= 32 else 1) if method == "rkc" else 48 if n_sp <= 32 else 16


def wide_lanes(n_sp: int) -> int:
    """Lanes per system of the wide variant: one species to a lane."""
    return 32 if n_sp <= 32 else 64


def _wide_layout(net, L, thermal=False):
    """The wide layout of a network (rk_group.hpp group_rhs_wide): lane r owns
    unknown r (species r; with the energy equation T, then the species), forms
    the rates at positions m L + r and adds its species' signed rates.  LDS area
    of a system (doubles): C [0, N), the place of lanes without a species at
    N + 1 | +q | the zero | scratch | -q, with -q a multiple of 64 behind +q (one
    instruction stores both)."""
    n, nr = net.n_sp, net.n_rx
    nu = n + 1 if thermal else n
    assert nu <= L
    R = -(-nr // L)
    pos_of, rx_of, m_first = _group_positions(net, L, R)
    off_q = n + 2 + (n % 2)
    off_zero = off_q + R * L
    off_red = off_zero + 1 + (off_zero + 1) % 2
    # with the energy equation two species rows follow the RKC recurrence's
    # coefficients, which stay in the scratch across evaluations
    off_e1 = off_red + GROUP_COEF_DOUBLES
    off_e2 = off_e1 + n + 1 + (n + 1) % 2
    red_len = max(nu + 1, off_e2 + n + 1 - off_red) if thermal else n
    neg = -(-(off_red + red_len - off_q) // 64) * 64
    lds = off_q + neg + R * L
    lds += lds % 2
    terms = [[(c >> 1, c & 1) for c in lst] for lst in _species_terms(net)]
    T = max(len(t) for t in terms)
    T += (-T) % 4
    first = nu - n
    seqs = [terms[r - first] if first <= r < nu else [] for r in range(L)]
    seqs = [q + [None] * (T - len(q)) for q in seqs]
    _spread_banks(net, L, R, m_first, pos_of, rx_of, seqs, neg, off_q, off_zero, lds)
    ops = []                     # [L][R][4] LDS byte offsets; [M]: byte offset of C_N
    for r in range(L):
        for m in range(R):
            j = rx_of[m * L + r]
            ops += [8 * (int(k) if k >= 0 else n) if j >= 0 else 0
                    for k in ((*net.reac[j], *net.prod[j]) if j >= 0 else (0,) * 4)]
    tm = [8 * (off_zero if e is None else off_q + pos_of[e[0]] + neg * e[1])
          for q in seqs for e in q]     # [L][T]
    return dict(n=n, nr=nr, nu=nu, L=L, R=R, m_first=m_first, off_q=off_q, off_zero=off_zero,
                off_red=off_red, off_e1=off_e1, off_e2=off_e2, red_len=red_len, neg=neg, lds=lds,
                ops=ops, tm=tm, T=T, rx_of=rx_of)


def wide_source(net, tag: str) -> str:
    """The wide variant of a network: one species per lane, for small batches."""
    n = net.n_sp
    G = _wide_layout(net, wide_lanes(n))
    return f"""
// Wide variant: {G["L"]} lanes per system, one species per lane (rk_group.hpp).
struct WNet {{
  static constexpr bool kWide = true;
  // largest batches it runs, in systems per SIMD (rk_group.hpp group_rhs_wide)
  static constexpr int kMaxRkck = {wide_limit(n, False, 'rkck')};
  static constexpr int kMaxRkc = {wide_limit(n, False, 'rkc')};
  static constexpr int N = {n};
  static constexpr int NR = {G["nr"]};
  static constexpr int kL = {G["L"]};
  static constexpr int kGroupLanes = {G["L"]};
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  static constexpr int kWavesPerEuRkc = {2 if n <= 32 else 1};
  static constexpr int kWavesPerEuRkck = 2;
  static constexpr int S = 1;
  static constexpr int R = {G["R"]};
  static constexpr int kMSlot = {G["m_first"]};   // first slot that may hold a [M] reaction
  static constexpr int kOffC = 0;
  static constexpr int kOffQ = {G["off_q"]};
  static constexpr int kOffZero = {G["off_zero"]};
  static constexpr int kNegOff = {G["neg"]};
  static constexpr int kOffRed = {G["off_red"]};
  static constexpr int kLdsPerSystem = {G["lds"]};
  static constexpr int kTermLen = {G["T"]};
  using Params = const double*;
{_table("kSp", "int", [r if r < n else -1 for r in range(G["L"])])}
{_table("kRxOf", "int16_t", G["rx_of"])}
  // LDS byte offsets within the system's area: each lane's rate operands
  // (R x 4), and the signed rates of its species in reaction order
{_table("kOp", "uint16_t", G["ops"], align=16)}
{_table("kTm", "uint16_t", G["tm"], align=16)}
  struct Lane {{
    double kf[R], kr[R];
    double W[S], iW[S];
    double rho, irho;
    uint32_t op[R][4], tm[kTermLen];   // LDS addresses, formed once per system
    uint32_t c_at;
  }};
  __device__ __attribute__((noinline)) static void rates(Params p, double T, double* lds, int r) {{
    const double lnT = crm::cr_log(T);
    double* const Q = lds + kOffQ;
#pragma nounroll
    for (int m = 0; m < R; ++m) {{
      const int j = kRxOf[m * kL + r];
      Q[m * kL + r] = j >= 0 ? crm::cr_exp(p[j] + p[NR + j] * lnT - p[2 * NR + j] / T) : 0.0;
    }}
  }}
  __device__ static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                              int64_t n, const Grp<WNet>& x) {{
    double* const Q = x.lds + kOffQ;
    rates(p, g[i], x.lds, x.r);
#pragma unroll
    for (int m = 0; m < R; ++m) {{
      const int j = kRxOf[m * kL + x.r];
      L.kf[m] = Q[m * kL + x.r];
      L.kr[m] = j >= 0 ? L.kf[m] * p[3 * NR + j] : 0.0;
    }}
    const int k = x.sp[0];
    L.W[0] = k >= 0 ? p[4 * NR + k] : 0.0;
    L.iW[0] = k >= 0 ? p[4 * NR + N + k] : 0.0;
    L.rho = g[n + i];
    L.irho = 1.0 / L.rho;
    const uint32_t base = lds_address(x.lds);
    L.c_at = base + 8 * (k >= 0 ? k : N + 1);
#pragma unroll
    for (int q = 0; q < 4 * R; ++q) L.op[q / 4][q % 4] = base + kOp[x.r * 4 * R + q];
#pragma unroll
    for (int t = 0; t < kTermLen; ++t) L.tm[t] = base + kTm[x.r * kTermLen + t];
    if (x.r == 0) x.lds[kOffZero] = 0.0;
  }}
}};
"""


def _vjp_source(net) -> str:
    """Vector-Jacobian products of the rate law, for the discrete adjoint:
    jtu = J(y)^T u and th += (df/dlnA)^T u.  With u~_k = (W_k / rho) u_k and
    r_j = sum_k nu_kj u~_k, both rate constants scale with A_j, so
    d(u^T f)/dlnA_j = r_j q_j; the concentrations take the adjoints of the
    products, [M] the adjoints of its factors, and (J^T u)_k =
    (rho / W_k) (C^_k + [M]^).  Same operations, same order, as the reference
    evaluation (products left to right, accumulators from zero)."""
    lines = []
    for j in range(net.n_rx):
        a, b = int(net.reac[j][0]), int(net.reac[j][1])
        c, d = int(net.prod[j][0]), int(net.prod[j][1])
        x = f"-uw[{b}]" if b >= 0 else "0.0"
        y = f"uw[{d}]" if d >= 0 else "0.0"
        lines.append(f"    r = ((-uw[{a}] + {x}) + uw[{c}]) + {y};")
        lines.append(f"    kf = L.kf[z + {j} * kLdsStride];")
        lines.append(f"    kr = kf * ld_uniform(iK, {j});")
        lines.append(f"    th[{j}] += r * ({_side('kf', net.reac[j])} - {_side('kr', net.prod[j])});")
        lines.append("    t = r * kf;")
        if b >= 0:
            lines.append(f"    Cb[{a}] += t * C[{b}];")
            lines.append(f"    Cb[{b}] += t * C[{a}];")
        else:
            lines.append(f"    Cb[{a}] += t * M;")
            lines.append(f"    Mb += t * C[{a}];")
        lines.append("    t = -r * kr;")
        if d >= 0:
            lines.append(f"    Cb[{c}] += t * C[{d}];")
            lines.append(f"    Cb[{d}] += t * C[{c}];")
        else:
            lines.append(f"    Cb[{c}] += t * M;")
            lines.append(f"    Mb += t * C[{c}];")
    body = "\n".join(lines)
    return f"""  static constexpr int kNTheta = NR;
  template <class VI, class VU, class VO>
  RKMI_HD static void vjp(const Lane& L, const Params& p, const VI& y, const VU& u, VO& jtu,
                          double (&th)[NR]) {{
    const double* __restrict__ iK = p + 3 * NR;
    const double* __restrict__ W = p + 4 * NR;
    const double* __restrict__ iW = W + N;
    double C[N], uw[N], Cb[N];
    const int z = opaque_zero();
#pragma unroll
    for (int k = 0; k < N; ++k) C[k] = (L.rho * y[k]) * ld_uniform(iW, k);
    double M = 0.0;
#pragma unroll
    for (int k = 0; k < N; ++k) M += C[k];
#pragma unroll
    for (int k = 0; k < N; ++k) uw[k] = (ld_uniform(W, k) * L.irho) * u[k];
#pragma unroll
    for (int k = 0; k < N; ++k) Cb[k] = 0.0;
    double Mb = 0.0;
    double r, kf, kr, t;
{body}
#pragma unroll
    for (int k = 0; k < N; ++k) jtu[k] = (L.rho * ld_uniform(iW, k)) * (Cb[k] + Mb);
  }}
"""


def _adjoint_exports(tag) -> str:
    return f"""
extern "C" int rkmi_gen_{tag}_taped(const rkmi::LaunchArgs* a, const rkmi::TapeArgs* t, void* s) {{
  return rkmi::launch_taped<rkmi::gen_{tag}::Net>(a, t, s);
}}

extern "C" int rkmi_gen_{tag}_taped_host(const rkmi::LaunchArgs* a, const rkmi::TapeArgs* t) {{
  return rkmi::host_taped<rkmi::gen_{tag}::Net>(a, t);
}}

extern "C" int rkmi_gen_{tag}_adjoint(const rkmi::AdjointArgs* a, void* s) {{
  return rkmi::launch_adjoint<rkmi::gen_{tag}::Net>(a, s);
}}

extern "C" int rkmi_gen_{tag}_adjoint_host(const rkmi::AdjointArgs* a) {{
  return rkmi::host_adjoint<rkmi::gen_{tag}::Net>(a);
}}
"""


def batch_source(tags, key: str) -> str:
    """One translation unit with the ragged-batch kernels over the networks
    `tags` (in this order)."""
    inc = "\n".join(f'#include "net_{t}.hpp"' for t in tags)
    nets = ", ".join(f"rkmi::gen_{t}::Net" for t in tags)
    return f"""// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Ragged batch over {len(tags)} networks: {", ".join(tags)}.
{inc}
#include "../rk_batch.hpp"

extern "C" int rkmi_batch_{key}_launch(const rkmi::BatchArgs* a, void* s) {{
  return rkmi::batch_launch<{nets}>(a, s);
}}

extern "C" int64_t rkmi_batch_{key}_workspace(const rkmi::BatchArgs* a) {{
  return rkmi::batch_workspace<{nets}>(a);
}}

extern "C" void rkmi_batch_{key}_free(void* cache) {{ rkmi::batch_free_cache(cache); }}
"""


def batch_key(tags) -> str:
    import hashlib
    return hashlib.sha1("/".join(tags).encode()).hexdigest()[:8]


def registry_source(entries, batches=(), thermal=()) -> str:
    """entries: list of (tag, net); batches: lists of tags compiled together;
    thermal: list of (tag, net) compiled with the energy equation."""
    decl, tabs, rows = [], [], []
    for tag, net in thermal:
        decl.append(f'extern "C" int rkmi_gen_{tag}_launch(const rkmi::LaunchArgs*, void*);')
        decl.append(f'extern "C" int rkmi_gen_{tag}_host(const rkmi::LaunchArgs*);')
        decl.append(f'extern "C" int64_t rkmi_gen_{tag}_workspace(int, int, int64_t);')
        if net.n_sp + 1 > REGISTER_SPECIES_LIMIT:
            decl.append(f"namespace rkmi {{ RateOrder gen_{tag}_rates(int); }}")
    for tag, net in entries:
        decl.append(f'extern "C" int rkmi_gen_{tag}_launch(const rkmi::LaunchArgs*, void*);')
        decl.append(f'extern "C" int rkmi_gen_{tag}_host(const rkmi::LaunchArgs*);')
        decl.append(f'extern "C" int64_t rkmi_gen_{tag}_workspace(int, int, int64_t);')
        if net.n_sp <= REGISTER_SPECIES_LIMIT:
            decl.append(f'extern "C" int rkmi_gen_{tag}_taped(const rkmi::LaunchArgs*, '
                        'const rkmi::TapeArgs*, void*);')
            decl.append(f'extern "C" int rkmi_gen_{tag}_taped_host(const rkmi::LaunchArgs*, '
                        'const rkmi::TapeArgs*);')
            decl.append(f'extern "C" int rkmi_gen_{tag}_adjoint(const rkmi::AdjointArgs*, void*);')
            decl.append(f'extern "C" int rkmi_gen_{tag}_adjoint_host(const rkmi::AdjointArgs*);')
            adj = (f"rkmi_gen_{tag}_taped, rkmi_gen_{tag}_taped_host, rkmi_gen_{tag}_adjoint, "
                   f"rkmi_gen_{tag}_adjoint_host")
        else:
            adj = "nullptr, nullptr, nullptr, nullptr"
        r = ", ".join(str(int(x)) for x in np.asarray(net.reac).reshape(-1))
        p = ", ".join(str(int(x)) for x in np.asarray(net.prod).reshape(-1))
        tabs.append(f"static const int32_t reac_{tag}[] = {{{r}}};")
        tabs.append(f"static const int32_t prod_{tag}[] = {{{p}}};")
        rows.append(f"    {{{net.n_sp}, {net.n_rx}, reac_{tag}, prod_{tag}, rkmi_gen_{tag}_launch, "
                    f"rkmi_gen_{tag}_host, rkmi_gen_{tag}_workspace, {adj}, 0, nullptr}},")
    index = {tag: k for k, (tag, _) in enumerate(entries)}
    for tag, net in thermal:
        base = tag[:-len(THERMAL_SUFFIX)]
        if f"static const int32_t reac_{base}[]" not in "\n".join(tabs):
            r = ", ".join(str(int(x)) for x in np.asarray(net.reac).reshape(-1))
            p = ", ".join(str(int(x)) for x in np.asarray(net.prod).reshape(-1))
            tabs.append(f"static const int32_t reac_{base}[] = {{{r}}};")
            tabs.append(f"static const int32_t prod_{base}[] = {{{p}}};")
        rows.append(f"    {{{net.n_sp}, {net.n_rx}, reac_{base}, prod_{base}, rkmi_gen_{tag}_launch, "
                    f"rkmi_gen_{tag}_host, rkmi_gen_{tag}_workspace, "
                    "nullptr, nullptr, nullptr, nullptr, 1, "
                    f"{f'gen_{tag}_rates' if net.n_sp + 1 > REGISTER_SPECIES_LIMIT else 'nullptr'}}},")
    brows = []
    for tags in batches:
        key = batch_key(tags)
        decl.append(f'extern "C" int rkmi_batch_{key}_launch(const rkmi::BatchArgs*, void*);')
        decl.append(f'extern "C" int64_t rkmi_batch_{key}_workspace(const rkmi::BatchArgs*);')
        decl.append(f'extern "C" void rkmi_batch_{key}_free(void*);')
        idx = ", ".join(str(index[t]) for t in tags)
        brows.append(f"    {{{len(tags)}, {{{idx}}}, rkmi_batch_{key}_launch, "
                     f"rkmi_batch_{key}_workspace, rkmi_batch_{key}_free}},")
    if not brows:
        brows.append("    {0, {0}, nullptr, nullptr, nullptr},")
    return (
        "// Generated by paper_1611_02274_amd/codegen.py -- do not edit.\n"
        "// Networks compiled into the library, matched by exact topology.\n"
        '#include "../rk_types.hpp"\n\n' + "\n".join(decl) + "\n\n" + "\n".join(tabs) +
        "\n\nnamespace rkmi {\nextern const GenEntry kGenRegistry[] = {\n" + "\n".join(rows) +
        "\n};\nextern const int kGenRegistrySize = " + str(len(rows)) + ";\n" +
        "extern const BatchEntry kBatchRegistry[] = {\n" + "\n".join(brows) + "\n};\n" +
        "extern const int kBatchRegistrySize = " + str(len(batches)) + ";\n"
        "}  // namespace rkmi\n")


def tag_of(net) -> str:
    return f"n{net.n_sp}r{net.n_rx}_{net.topology_key()[:8]}"


THERMAL_SUFFIX = "_th"


def generate(nets, out_dir: str = GEN_DIR, batches=(), thermal=()) -> list[str]:
    """Writes one source per network, one per batch (lists of networks compiled
    together), one per network compiled with the energy equation (`thermal`)
    and the registry; returns the paths of the sources to compile.  Files
    whose content is unchanged are left untouched."""
    os.makedirs(out_dir, exist_ok=True)
    paths, entries, tentries = [], [], []
    keep = set()
    for net in thermal:
        tag = tag_of(net) + THERMAL_SUFFIX
        tentries.append((tag, net))
        header, source = (thermal_source(net, tag) if net.n_sp + 1 <= REGISTER_SPECIES_LIMIT
                          else thermal_group_source(net, tag))
        keep.add(os.path.basename(_write(os.path.join(out_dir, f"net_{tag}.hpp"), header)))
        paths.append(_write(os.path.join(out_dir, f"net_{tag}.hip"), source))
    for net in nets:
        tag = tag_of(net)
        entries.append((tag, net))
        header, source = rhs_source(net, tag)
        keep.add(os.path.basename(_write(os.path.join(out_dir, f"net_{tag}.hpp"), header)))
        paths.append(_write(os.path.join(out_dir, f"net_{tag}.hip"), source))
    btags = [[tag_of(n) for n in b] for b in batches]
    for tags in btags:
        paths.append(_write(os.path.join(out_dir, f"batch_{batch_key(tags)}.hip"),
                            batch_source(tags, batch_key(tags))))
    paths.append(_write(os.path.join(out_dir, "registry.cpp"),
                        registry_source(entries, btags, tentries)))
    keep |= {os.path.basename(p) for p in paths}
    for f in os.listdir(out_dir):
        if f not in keep and f.startswith(("net_", "registry.", "batch_")):
            os.remove(os.path.join(out_dir, f))
    return paths


def _write(path: str, text: str) -> str:
    if os.path.exists(path):
        with open(path) as fh:
            if fh.read() == text:
                return path
    with open(path, "w") as fh:
        fh.write(text)
    return path


def standard_nets():
    from .inputs import standard_network
    return [standard_network(k) for k in (9, 13, 32, 53)]
