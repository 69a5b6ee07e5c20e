// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Mass-action network with the energy equation: 13 species + T, 27 reversible
// reactions (topology n13r27_7b5c2807_th).
#pragma once

#include "../rk_launch.hpp"

namespace rkmi {
namespace gen_n13r27_7b5c2807_th {

struct Net {
  static constexpr int NS = 13;
  static constexpr int N = NS + 1;
  static constexpr int NR = 27;
  // vectors in registers; k_f,j(T) of the current evaluation in the lane's LDS
  // slot, read back at an offset the optimizer cannot see through
  static constexpr bool kColumns = false;
  static constexpr int kGroupLanes = 1;
  static constexpr int kLaneDoubles = NR;
  static constexpr int kWavesPerEu = 2;
  static constexpr bool kExpTable = true;
  // uniform data: [lnA | beta | Ea | 1/K | W | 1/W | u0 | cv0 | cv1]
  using Params = const double*;
  struct Lane {
    double* kf;
    crm::ExpTable et;
    double rho, irho;
  };
  RKMI_HD static void init(Lane& L, const Params&, const double* __restrict__ g, int64_t i,
                           int64_t, double* slot) {
    L.kf = slot;
    L.et.p = shared_area<Net>(slot);
    L.rho = g[i];
    L.irho = 1.0 / L.rho;
  }
  template <class VI, class VO>
  RKMI_HD static void rhs(const Lane& L, const Params& p, const VI& y, VO& f) {
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
    // 3 exponentials side by side without a branch, their tables in LDS: one at a
    // time, each waited out its table reads and its own chain of operations (9
    // species 65536 systems 178 -> 114 ms, 13 species 84 -> 54 ms)
#pragma nounroll
    for (int j0 = 0; j0 < NR; j0 += 3) {
      double a[3], e[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int j = j0 + k < NR ? j0 + k : NR - 1;
        a[k] = ld_uniform(p, j) + ld_uniform(p, NR + j) * lnT - ld_uniform(p, 2 * NR + j) * invT;
      }
      crm::cr_exp_n<3>(a, e, L.et);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        L.kf[z + (j0 + k < NR ? j0 + k : NR - 1) * kLdsStride] = e[k];
    }
    double C[NS], om[NS];
#pragma unroll
    for (int k = 0; k < NS; ++k) C[k] = (L.rho * y[1 + k]) * ld_uniform(iW, k);
    double M = 0.0;
#pragma unroll
    for (int k = 0; k < NS; ++k) M += C[k];
#pragma unroll
    for (int k = 0; k < NS; ++k) om[k] = 0.0;
    double q, kf, kr;
    kf = L.kf[z + 0 * kLdsStride];
    kr = kf * ld_uniform(iK, 0);
    q = (kf * C[3]) * C[5] - (kr * C[0]) * C[6];
    om[3] -= q;
    om[5] -= q;
    om[0] += q;
    om[6] += q;
    kf = L.kf[z + 1 * kLdsStride];
    kr = kf * ld_uniform(iK, 1);
    q = (kf * C[0]) * C[5] - (kr * C[3]) * C[8];
    om[0] -= q;
    om[5] -= q;
    om[3] += q;
    om[8] += q;
    kf = L.kf[z + 2 * kLdsStride];
    kr = kf * ld_uniform(iK, 2);
    q = (kf * C[3]) * C[8] - (kr * C[6]) * M;
    om[3] -= q;
    om[8] -= q;
    om[6] += q;
    kf = L.kf[z + 3 * kLdsStride];
    kr = kf * ld_uniform(iK, 3);
    q = (kf * C[1]) * C[5] - (kr * C[8]) * C[10];
    om[1] -= q;
    om[5] -= q;
    om[8] += q;
    om[10] += q;
    kf = L.kf[z + 4 * kLdsStride];
    kr = kf * ld_uniform(iK, 4);
    q = (kf * C[0]) * C[9] - (kr * C[6]) * C[8];
    om[0] -= q;
    om[9] -= q;
    om[6] += q;
    om[8] += q;
    kf = L.kf[z + 5 * kLdsStride];
    kr = kf * ld_uniform(iK, 5);
    q = (kf * C[4]) * C[8] - (kr * C[3]) * C[5];
    om[4] -= q;
    om[8] -= q;
    om[3] += q;
    om[5] += q;
    kf = L.kf[z + 6 * kLdsStride];
    kr = kf * ld_uniform(iK, 6);
    q = (kf * C[9]) * M - (kr * C[5]) * C[8];
    om[9] -= q;
    om[5] += q;
    om[8] += q;
    kf = L.kf[z + 7 * kLdsStride];
    kr = kf * ld_uniform(iK, 7);
    q = (kf * C[6]) * C[6] - (kr * C[4]) * C[9];
    om[6] -= q;
    om[6] -= q;
    om[4] += q;
    om[9] += q;
    kf = L.kf[z + 8 * kLdsStride];
    kr = kf * ld_uniform(iK, 8);
    q = (kf * C[6]) * M - (kr * C[2]) * C[4];
    om[6] -= q;
    om[2] += q;
    om[4] += q;
    kf = L.kf[z + 9 * kLdsStride];
    kr = kf * ld_uniform(iK, 9);
    q = (kf * C[2]) * C[3] - (kr * C[5]) * M;
    om[2] -= q;
    om[3] -= q;
    om[5] += q;
    kf = L.kf[z + 10 * kLdsStride];
    kr = kf * ld_uniform(iK, 10);
    q = (kf * C[0]) * C[5] - (kr * C[2]) * C[4];
    om[0] -= q;
    om[5] -= q;
    om[2] += q;
    om[4] += q;
    kf = L.kf[z + 11 * kLdsStride];
    kr = kf * ld_uniform(iK, 11);
    q = (kf * C[0]) * C[8] - (kr * C[5]) * M;
    om[0] -= q;
    om[8] -= q;
    om[5] += q;
    kf = L.kf[z + 12 * kLdsStride];
    kr = kf * ld_uniform(iK, 12);
    q = (kf * C[7]) * C[12] - (kr * C[2]) * C[11];
    om[7] -= q;
    om[12] -= q;
    om[2] += q;
    om[11] += q;
    kf = L.kf[z + 13 * kLdsStride];
    kr = kf * ld_uniform(iK, 13);
    q = (kf * C[0]) * C[2] - (kr * C[8]) * M;
    om[0] -= q;
    om[2] -= q;
    om[8] += q;
    kf = L.kf[z + 14 * kLdsStride];
    kr = kf * ld_uniform(iK, 14);
    q = (kf * C[9]) * M - (kr * C[2]) * C[6];
    om[9] -= q;
    om[2] += q;
    om[6] += q;
    kf = L.kf[z + 15 * kLdsStride];
    kr = kf * ld_uniform(iK, 15);
    q = (kf * C[4]) * C[8] - (kr * C[0]) * C[6];
    om[4] -= q;
    om[8] -= q;
    om[0] += q;
    om[6] += q;
    kf = L.kf[z + 16 * kLdsStride];
    kr = kf * ld_uniform(iK, 16);
    q = (kf * C[6]) * C[8] - (kr * C[5]) * C[5];
    om[6] -= q;
    om[8] -= q;
    om[5] += q;
    om[5] += q;
    kf = L.kf[z + 17 * kLdsStride];
    kr = kf * ld_uniform(iK, 17);
    q = (kf * C[0]) * C[7] - (kr * C[1]) * C[10];
    om[0] -= q;
    om[7] -= q;
    om[1] += q;
    om[10] += q;
    kf = L.kf[z + 18 * kLdsStride];
    kr = kf * ld_uniform(iK, 18);
    q = (kf * C[4]) * M - (kr * C[0]) * C[3];
    om[4] -= q;
    om[0] += q;
    om[3] += q;
    kf = L.kf[z + 19 * kLdsStride];
    kr = kf * ld_uniform(iK, 19);
    q = (kf * C[0]) * C[9] - (kr * C[5]) * C[5];
    om[0] -= q;
    om[9] -= q;
    om[5] += q;
    om[5] += q;
    kf = L.kf[z + 20 * kLdsStride];
    kr = kf * ld_uniform(iK, 20);
    q = (kf * C[10]) * C[10] - (kr * C[3]) * C[7];
    om[10] -= q;
    om[10] -= q;
    om[3] += q;
    om[7] += q;
    kf = L.kf[z + 21 * kLdsStride];
    kr = kf * ld_uniform(iK, 21);
    q = (kf * C[4]) * C[5] - (kr * C[3]) * C[6];
    om[4] -= q;
    om[5] -= q;
    om[3] += q;
    om[6] += q;
    kf = L.kf[z + 22 * kLdsStride];
    kr = kf * ld_uniform(iK, 22);
    q = (kf * C[0]) * C[10] - (kr * C[1]) * C[3];
    om[0] -= q;
    om[10] -= q;
    om[1] += q;
    om[3] += q;
    kf = L.kf[z + 23 * kLdsStride];
    kr = kf * ld_uniform(iK, 23);
    q = (kf * C[1]) * C[8] - (kr * C[2]) * C[10];
    om[1] -= q;
    om[8] -= q;
    om[2] += q;
    om[10] += q;
    kf = L.kf[z + 24 * kLdsStride];
    kr = kf * ld_uniform(iK, 24);
    q = (kf * C[8]) * C[8] - (kr * C[2]) * C[5];
    om[8] -= q;
    om[8] -= q;
    om[2] += q;
    om[5] += q;
    kf = L.kf[z + 25 * kLdsStride];
    kr = kf * ld_uniform(iK, 25);
    q = (kf * C[2]) * C[9] - (kr * C[12]) * M;
    om[2] -= q;
    om[9] -= q;
    om[12] += q;
    kf = L.kf[z + 26 * kLdsStride];
    kr = kf * ld_uniform(iK, 26);
    q = (kf * C[5]) * C[6] - (kr * C[3]) * C[9];
    om[5] -= q;
    om[6] -= q;
    om[3] += q;
    om[9] += q;
#pragma unroll
    for (int k = 0; k < NS; ++k) f[1 + k] = (ld_uniform(W, k) * om[k]) * L.irho;
    double sum = 0.0, cv = 0.0;
#pragma unroll
    for (int k = 0; k < NS; ++k) {
      const double e = ld_uniform(u0, k) + (ld_uniform(cv0, k) + ld_uniform(cv1, k) * T) * T;
      sum += (e * om[k]) * ld_uniform(W, k);
      cv += y[1 + k] * (ld_uniform(cv0, k) + 2.0 * ld_uniform(cv1, k) * T);
    }
    f[0] = -((sum * L.irho) / cv);
  }
};

// Batches of at most one wave per SIMD: the wave has the SIMD's registers to
// itself.
struct NetR : Net {
  static constexpr int kWavesPerEu = 1;
};

}  // namespace gen_n13r27_7b5c2807_th

template <>
struct SparseVariant<gen_n13r27_7b5c2807_th::Net> {
  using type = gen_n13r27_7b5c2807_th::NetR;
};

}  // namespace rkmi
