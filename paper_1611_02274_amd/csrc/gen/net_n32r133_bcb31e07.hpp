// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Mass-action network: 32 species, 133 reversible reactions (topology n32r133_bcb31e07).
#pragma once

#include "../rk_adjoint.hpp"
#include "../rk_group.hpp"

namespace rkmi {
namespace gen_n32r133_bcb31e07 {

struct Net {
  static constexpr int N = 32;
  static constexpr int NR = 133;
  // vectors and the forward rate constants k_f,j of the system live in slot
  // columns (stride kLdsStride); each k_f,j is read once per evaluation
  static constexpr bool kColumns = true;
  static constexpr int kGroupLanes = 1;
  static constexpr int kLaneDoubles = NR;
  using Params = const double*;
  struct Lane {
    const double* kf;
    double rho, irho;
  };
  RKMI_HD static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                           int64_t n, double* slot) {
    const double T = g[i];
    const double rho = g[n + i];
    const double lnT = crm::cr_log(T);
    for (int j = 0; j < NR; ++j)
      slot[j * kLdsStride] = crm::cr_exp(p[j] + p[NR + j] * lnT - p[2 * NR + j] / T);
    L.kf = slot;
    L.rho = rho;
    L.irho = 1.0 / rho;
  }
  template <class VI, class VO>
  RKMI_HD static void rhs(const Lane& L, const Params& p, const VI& y, VO& f) {
    const double* __restrict__ iK = p + 3 * NR;
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
    kf = L.kf[0 * kLdsStride];
    kr = kf * ld_uniform(iK, 0);
    q = (kf * C[8]) * C[15] - (kr * C[4]) * C[23];
    om[8] -= q;
    om[15] -= q;
    om[4] += q;
    om[23] += q;
    kf = L.kf[1 * kLdsStride];
    kr = kf * ld_uniform(iK, 1);
    q = (kf * C[15]) * C[30] - (kr * C[6]) * C[7];
    om[15] -= q;
    om[30] -= q;
    om[6] += q;
    om[7] += q;
    kf = L.kf[2 * kLdsStride];
    kr = kf * ld_uniform(iK, 2);
    q = (kf * C[12]) * C[28] - (kr * C[17]) * C[17];
    om[12] -= q;
    om[28] -= q;
    om[17] += q;
    om[17] += q;
    kf = L.kf[3 * kLdsStride];
    kr = kf * ld_uniform(iK, 3);
    q = (kf * C[22]) * C[23] - (kr * C[4]) * C[27];
    om[22] -= q;
    om[23] -= q;
    om[4] += q;
    om[27] += q;
    kf = L.kf[4 * kLdsStride];
    kr = kf * ld_uniform(iK, 4);
    q = (kf * C[9]) * C[25] - (kr * C[23]) * C[27];
    om[9] -= q;
    om[25] -= q;
    om[23] += q;
    om[27] += q;
    kf = L.kf[5 * kLdsStride];
    kr = kf * ld_uniform(iK, 5);
    q = (kf * C[6]) * C[21] - (kr * C[14]) * C[19];
    om[6] -= q;
    om[21] -= q;
    om[14] += q;
    om[19] += q;
    kf = L.kf[6 * kLdsStride];
    kr = kf * ld_uniform(iK, 6);
    q = (kf * C[10]) * C[21] - (kr * C[3]) * C[26];
    om[10] -= q;
    om[21] -= q;
    om[3] += q;
    om[26] += q;
    kf = L.kf[7 * kLdsStride];
    kr = kf * ld_uniform(iK, 7);
    q = (kf * C[3]) * C[26] - (kr * C[13]) * C[28];
    om[3] -= q;
    om[26] -= q;
    om[13] += q;
    om[28] += q;
    kf = L.kf[8 * kLdsStride];
    kr = kf * ld_uniform(iK, 8);
    q = (kf * C[26]) * C[28] - (kr * C[21]) * C[25];
    om[26] -= q;
    om[28] -= q;
    om[21] += q;
    om[25] += q;
    kf = L.kf[9 * kLdsStride];
    kr = kf * ld_uniform(iK, 9);
    q = (kf * C[8]) * C[21] - (kr * C[5]) * C[9];
    om[8] -= q;
    om[21] -= q;
    om[5] += q;
    om[9] += q;
    kf = L.kf[10 * kLdsStride];
    kr = kf * ld_uniform(iK, 10);
    q = (kf * C[11]) * C[14] - (kr * C[2]) * C[24];
    om[11] -= q;
    om[14] -= q;
    om[2] += q;
    om[24] += q;
    kf = L.kf[11 * kLdsStride];
    kr = kf * ld_uniform(iK, 11);
    q = (kf * C[9]) * C[16] - (kr * C[7]) * C[25];
    om[9] -= q;
    om[16] -= q;
    om[7] += q;
    om[25] += q;
    kf = L.kf[12 * kLdsStride];
    kr = kf * ld_uniform(iK, 12);
    q = (kf * C[9]) * C[24] - (kr * C[18]) * C[28];
    om[9] -= q;
    om[24] -= q;
    om[18] += q;
    om[28] += q;
    kf = L.kf[13 * kLdsStride];
    kr = kf * ld_uniform(iK, 13);
    q = (kf * C[11]) * C[17] - (kr * C[5]) * C[13];
    om[11] -= q;
    om[17] -= q;
    om[5] += q;
    om[13] += q;
    kf = L.kf[14 * kLdsStride];
    kr = kf * ld_uniform(iK, 14);
    q = (kf * C[1]) * C[22] - (kr * C[2]) * C[21];
    om[1] -= q;
    om[22] -= q;
    om[2] += q;
    om[21] += q;
    kf = L.kf[15 * kLdsStride];
    kr = kf * ld_uniform(iK, 15);
    q = (kf * C[16]) * C[21] - (kr * C[14]) * C[25];
    om[16] -= q;
    om[21] -= q;
    om[14] += q;
    om[25] += q;
    kf = L.kf[16 * kLdsStride];
    kr = kf * ld_uniform(iK, 16);
    q = (kf * C[7]) * C[20] - (kr * C[10]) * C[28];
    om[7] -= q;
    om[20] -= q;
    om[10] += q;
    om[28] += q;
    kf = L.kf[17 * kLdsStride];
    kr = kf * ld_uniform(iK, 17);
    q = (kf * C[2]) * C[2] - (kr * C[11]) * M;
    om[2] -= q;
    om[2] -= q;
    om[11] += q;
    kf = L.kf[18 * kLdsStride];
    kr = kf * ld_uniform(iK, 18);
    q = (kf * C[27]) * M - (kr * C[6]) * C[21];
    om[27] -= q;
    om[6] += q;
    om[21] += q;
    kf = L.kf[19 * kLdsStride];
    kr = kf * ld_uniform(iK, 19);
    q = (kf * C[16]) * C[21] - (kr * C[17]) * C[20];
    om[16] -= q;
    om[21] -= q;
    om[17] += q;
    om[20] += q;
    kf = L.kf[20 * kLdsStride];
    kr = kf * ld_uniform(iK, 20);
    q = (kf * C[24]) * C[31] - (kr * C[20]) * C[22];
    om[24] -= q;
    om[31] -= q;
    om[20] += q;
    om[22] += q;
    kf = L.kf[21 * kLdsStride];
    kr = kf * ld_uniform(iK, 21);
    q = (kf * C[20]) * C[21] - (kr * C[3]) * C[17];
    om[20] -= q;
    om[21] -= q;
    om[3] += q;
    om[17] += q;
    kf = L.kf[22 * kLdsStride];
    kr = kf * ld_uniform(iK, 22);
    q = (kf * C[9]) * C[29] - (kr * C[18]) * C[20];
    om[9] -= q;
    om[29] -= q;
    om[18] += q;
    om[20] += q;
    kf = L.kf[23 * kLdsStride];
    kr = kf * ld_uniform(iK, 23);
    q = (kf * C[10]) * C[28] - (kr * C[14]) * C[19];
    om[10] -= q;
    om[28] -= q;
    om[14] += q;
    om[19] += q;
    kf = L.kf[24 * kLdsStride];
    kr = kf * ld_uniform(iK, 24);
    q = (kf * C[4]) * C[17] - (kr * C[5]) * C[7];
    om[4] -= q;
    om[17] -= q;
    om[5] += q;
    om[7] += q;
    kf = L.kf[25 * kLdsStride];
    kr = kf * ld_uniform(iK, 25);
    q = (kf * C[22]) * M - (kr * C[3]) * C[14];
    om[22] -= q;
    om[3] += q;
    om[14] += q;
    kf = L.kf[26 * kLdsStride];
    kr = kf * ld_uniform(iK, 26);
    q = (kf * C[24]) * C[27] - (kr * C[12]) * C[14];
    om[24] -= q;
    om[27] -= q;
    om[12] += q;
    om[14] += q;
    kf = L.kf[27 * kLdsStride];
    kr = kf * ld_uniform(iK, 27);
    q = (kf * C[0]) * C[26] - (kr * C[2]) * C[9];
    om[0] -= q;
    om[26] -= q;
    om[2] += q;
    om[9] += q;
    kf = L.kf[28 * kLdsStride];
    kr = kf * ld_uniform(iK, 28);
    q = (kf * C[1]) * C[9] - (kr * C[15]) * C[25];
    om[1] -= q;
    om[9] -= q;
    om[15] += q;
    om[25] += q;
    kf = L.kf[29 * kLdsStride];
    kr = kf * ld_uniform(iK, 29);
    q = (kf * C[9]) * C[15] - (kr * C[19]) * C[28];
    om[9] -= q;
    om[15] -= q;
    om[19] += q;
    om[28] += q;
    kf = L.kf[30 * kLdsStride];
    kr = kf * ld_uniform(iK, 30);
    q = (kf * C[20]) * C[26] - (kr * C[8]) * C[13];
    om[20] -= q;
    om[26] -= q;
    om[8] += q;
    om[13] += q;
    kf = L.kf[31 * kLdsStride];
    kr = kf * ld_uniform(iK, 31);
    q = (kf * C[23]) * C[31] - (kr * C[19]) * C[28];
    om[23] -= q;
    om[31] -= q;
    om[19] += q;
    om[28] += q;
    kf = L.kf[32 * kLdsStride];
    kr = kf * ld_uniform(iK, 32);
    q = (kf * C[10]) * C[21] - (kr * C[15]) * C[18];
    om[10] -= q;
    om[21] -= q;
    om[15] += q;
    om[18] += q;
    kf = L.kf[33 * kLdsStride];
    kr = kf * ld_uniform(iK, 33);
    q = (kf * C[14]) * C[25] - (kr * C[23]) * C[24];
    om[14] -= q;
    om[25] -= q;
    om[23] += q;
    om[24] += q;
    kf = L.kf[34 * kLdsStride];
    kr = kf * ld_uniform(iK, 34);
    q = (kf * C[6]) * C[18] - (kr * C[7]) * C[13];
    om[6] -= q;
    om[18] -= q;
    om[7] += q;
    om[13] += q;
    kf = L.kf[35 * kLdsStride];
    kr = kf * ld_uniform(iK, 35);
    q = (kf * C[2]) * C[26] - (kr * C[13]) * C[31];
    om[2] -= q;
    om[26] -= q;
    om[13] += q;
    om[31] += q;
    kf = L.kf[36 * kLdsStride];
    kr = kf * ld_uniform(iK, 36);
    q = (kf * C[3]) * C[22] - (kr * C[14]) * C[14];
    om[3] -= q;
    om[22] -= q;
    om[14] += q;
    om[14] += q;
    kf = L.kf[37 * kLdsStride];
    kr = kf * ld_uniform(iK, 37);
    q = (kf * C[16]) * C[26] - (kr * C[6]) * C[12];
    om[16] -= q;
    om[26] -= q;
    om[6] += q;
    om[12] += q;
    kf = L.kf[38 * kLdsStride];
    kr = kf * ld_uniform(iK, 38);
    q = (kf * C[1]) * C[26] - (kr * C[16]) * C[16];
    om[1] -= q;
    om[26] -= q;
    om[16] += q;
    om[16] += q;
    kf = L.kf[39 * kLdsStride];
    kr = kf * ld_uniform(iK, 39);
    q = (kf * C[5]) * C[13] - (kr * C[10]) * C[22];
    om[5] -= q;
    om[13] -= q;
    om[10] += q;
    om[22] += q;
    kf = L.kf[40 * kLdsStride];
    kr = kf * ld_uniform(iK, 40);
    q = (kf * C[2]) * C[28] - (kr * C[14]) * C[15];
    om[2] -= q;
    om[28] -= q;
    om[14] += q;
    om[15] += q;
    kf = L.kf[41 * kLdsStride];
    kr = kf * ld_uniform(iK, 41);
    q = (kf * C[13]) * C[28] - (kr * C[19]) * C[24];
    om[13] -= q;
    om[28] -= q;
    om[19] += q;
    om[24] += q;
    kf = L.kf[42 * kLdsStride];
    kr = kf * ld_uniform(iK, 42);
    q = (kf * C[26]) * C[27] - (kr * C[12]) * C[25];
    om[26] -= q;
    om[27] -= q;
    om[12] += q;
    om[25] += q;
    kf = L.kf[43 * kLdsStride];
    kr = kf * ld_uniform(iK, 43);
    q = (kf * C[16]) * C[24] - (kr * C[10]) * C[22];
    om[16] -= q;
    om[24] -= q;
    om[10] += q;
    om[22] += q;
    kf = L.kf[44 * kLdsStride];
    kr = kf * ld_uniform(iK, 44);
    q = (kf * C[10]) * C[31] - (kr * C[16]) * C[20];
    om[10] -= q;
    om[31] -= q;
    om[16] += q;
    om[20] += q;
    kf = L.kf[45 * kLdsStride];
    kr = kf * ld_uniform(iK, 45);
    q = (kf * C[4]) * C[30] - (kr * C[1]) * C[17];
    om[4] -= q;
    om[30] -= q;
    om[1] += q;
    om[17] += q;
    kf = L.kf[46 * kLdsStride];
    kr = kf * ld_uniform(iK, 46);
    q = (kf * C[18]) * C[19] - (kr * C[6]) * C[12];
    om[18] -= q;
    om[19] -= q;
    om[6] += q;
    om[12] += q;
    kf = L.kf[47 * kLdsStride];
    kr = kf * ld_uniform(iK, 47);
    q = (kf * C[3]) * C[7] - (kr * C[2]) * C[8];
    om[3] -= q;
    om[7] -= q;
    om[2] += q;
    om[8] += q;
    kf = L.kf[48 * kLdsStride];
    kr = kf * ld_uniform(iK, 48);
    q = (kf * C[10]) * C[21] - (kr * C[14]) * C[30];
    om[10] -= q;
    om[21] -= q;
    om[14] += q;
    om[30] += q;
    kf = L.kf[49 * kLdsStride];
    kr = kf * ld_uniform(iK, 49);
    q = (kf * C[4]) * C[16] - (kr * C[20]) * C[31];
    om[4] -= q;
    om[16] -= q;
    om[20] += q;
    om[31] += q;
    kf = L.kf[50 * kLdsStride];
    kr = kf * ld_uniform(iK, 50);
    q = (kf * C[19]) * C[22] - (kr * C[14]) * C[25];
    om[19] -= q;
    om[22] -= q;
    om[14] += q;
    om[25] += q;
    kf = L.kf[51 * kLdsStride];
    kr = kf * ld_uniform(iK, 51);
    q = (kf * C[1]) * C[27] - (kr * C[6]) * C[17];
    om[1] -= q;
    om[27] -= q;
    om[6] += q;
    om[17] += q;
    kf = L.kf[52 * kLdsStride];
    kr = kf * ld_uniform(iK, 52);
    q = (kf * C[5]) * C[14] - (kr * C[4]) * C[22];
    om[5] -= q;
    om[14] -= q;
    om[4] += q;
    om[22] += q;
    kf = L.kf[53 * kLdsStride];
    kr = kf * ld_uniform(iK, 53);
    q = (kf * C[14]) * C[23] - (kr * C[8]) * C[20];
    om[14] -= q;
    om[23] -= q;
    om[8] += q;
    om[20] += q;
    kf = L.kf[54 * kLdsStride];
    kr = kf * ld_uniform(iK, 54);
    q = (kf * C[20]) * C[27] - (kr * C[21]) * C[30];
    om[20] -= q;
    om[27] -= q;
    om[21] += q;
    om[30] += q;
    kf = L.kf[55 * kLdsStride];
    kr = kf * ld_uniform(iK, 55);
    q = (kf * C[22]) * C[30] - (kr * C[18]) * C[31];
    om[22] -= q;
    om[30] -= q;
    om[18] += q;
    om[31] += q;
    kf = L.kf[56 * kLdsStride];
    kr = kf * ld_uniform(iK, 56);
    q = (kf * C[3]) * C[27] - (kr * C[17]) * C[20];
    om[3] -= q;
    om[27] -= q;
    om[17] += q;
    om[20] += q;
    kf = L.kf[57 * kLdsStride];
    kr = kf * ld_uniform(iK, 57);
    q = (kf * C[5]) * C[12] - (kr * C[22]) * C[27];
    om[5] -= q;
    om[12] -= q;
    om[22] += q;
    om[27] += q;
    kf = L.kf[58 * kLdsStride];
    kr = kf * ld_uniform(iK, 58);
    q = (kf * C[3]) * C[26] - (kr * C[12]) * M;
    om[3] -= q;
    om[26] -= q;
    om[12] += q;
    kf = L.kf[59 * kLdsStride];
    kr = kf * ld_uniform(iK, 59);
    q = (kf * C[15]) * C[22] - (kr * C[5]) * C[20];
    om[15] -= q;
    om[22] -= q;
    om[5] += q;
    om[20] += q;
    kf = L.kf[60 * kLdsStride];
    kr = kf * ld_uniform(iK, 60);
    q = (kf * C[20]) * C[31] - (kr * C[3]) * C[7];
    om[20] -= q;
    om[31] -= q;
    om[3] += q;
    om[7] += q;
    kf = L.kf[61 * kLdsStride];
    kr = kf * ld_uniform(iK, 61);
    q = (kf * C[15]) * C[20] - (kr * C[4]) * C[6];
    om[15] -= q;
    om[20] -= q;
    om[4] += q;
    om[6] += q;
    kf = L.kf[62 * kLdsStride];
    kr = kf * ld_uniform(iK, 62);
    q = (kf * C[23]) * C[30] - (kr * C[19]) * C[25];
    om[23] -= q;
    om[30] -= q;
    om[19] += q;
    om[25] += q;
    kf = L.kf[63 * kLdsStride];
    kr = kf * ld_uniform(iK, 63);
    q = (kf * C[25]) * C[25] - (kr * C[9]) * C[30];
    om[25] -= q;
    om[25] -= q;
    om[9] += q;
    om[30] += q;
    kf = L.kf[64 * kLdsStride];
    kr = kf * ld_uniform(iK, 64);
    q = (kf * C[15]) * C[21] - (kr * C[3]) * C[8];
    om[15] -= q;
    om[21] -= q;
    om[3] += q;
    om[8] += q;
    kf = L.kf[65 * kLdsStride];
    kr = kf * ld_uniform(iK, 65);
    q = (kf * C[28]) * C[31] - (kr * C[4]) * C[8];
    om[28] -= q;
    om[31] -= q;
    om[4] += q;
    om[8] += q;
    kf = L.kf[66 * kLdsStride];
    kr = kf * ld_uniform(iK, 66);
    q = (kf * C[2]) * C[25] - (kr * C[26]) * M;
    om[2] -= q;
    om[25] -= q;
    om[26] += q;
    kf = L.kf[67 * kLdsStride];
    kr = kf * ld_uniform(iK, 67);
    q = (kf * C[7]) * C[11] - (kr * C[4]) * C[13];
    om[7] -= q;
    om[11] -= q;
    om[4] += q;
    om[13] += q;
    kf = L.kf[68 * kLdsStride];
    kr = kf * ld_uniform(iK, 68);
    q = (kf * C[9]) * C[29] - (kr * C[13]) * C[21];
    om[9] -= q;
    om[29] -= q;
    om[13] += q;
    om[21] += q;
    kf = L.kf[69 * kLdsStride];
    kr = kf * ld_uniform(iK, 69);
    q = (kf * C[4]) * C[7] - (kr * C[20]) * C[28];
    om[4] -= q;
    om[7] -= q;
    om[20] += q;
    om[28] += q;
    kf = L.kf[70 * kLdsStride];
    kr = kf * ld_uniform(iK, 70);
    q = (kf * C[3]) * C[26] - (kr * C[9]) * C[11];
    om[3] -= q;
    om[26] -= q;
    om[9] += q;
    om[11] += q;
    kf = L.kf[71 * kLdsStride];
    kr = kf * ld_uniform(iK, 71);
    q = (kf * C[14]) * C[23] - (kr * C[15]) * C[17];
    om[14] -= q;
    om[23] -= q;
    om[15] += q;
    om[17] += q;
    kf = L.kf[72 * kLdsStride];
    kr = kf * ld_uniform(iK, 72);
    q = (kf * C[3]) * C[31] - (kr * C[2]) * C[28];
    om[3] -= q;
    om[31] -= q;
    om[2] += q;
    om[28] += q;
    kf = L.kf[73 * kLdsStride];
    kr = kf * ld_uniform(iK, 73);
    q = (kf * C[8]) * C[26] - (kr * C[17]) * C[25];
    om[8] -= q;
    om[26] -= q;
    om[17] += q;
    om[25] += q;
    kf = L.kf[74 * kLdsStride];
    kr = kf * ld_uniform(iK, 74);
    q = (kf * C[1]) * C[21] - (kr * C[4]) * C[16];
    om[1] -= q;
    om[21] -= q;
    om[4] += q;
    om[16] += q;
    kf = L.kf[75 * kLdsStride];
    kr = kf * ld_uniform(iK, 75);
    q = (kf * C[4]) * C[30] - (kr * C[3]) * C[25];
    om[4] -= q;
    om[30] -= q;
    om[3] += q;
    om[25] += q;
    kf = L.kf[76 * kLdsStride];
    kr = kf * ld_uniform(iK, 76);
    q = (kf * C[7]) * C[22] - (kr * C[14]) * C[17];
    om[7] -= q;
    om[22] -= q;
    om[14] += q;
    om[17] += q;
    kf = L.kf[77 * kLdsStride];
    kr = kf * ld_uniform(iK, 77);
    q = (kf * C[16]) * M - (kr * C[0]) * C[10];
    om[16] -= q;
    om[0] += q;
    om[10] += q;
    kf = L.kf[78 * kLdsStride];
    kr = kf * ld_uniform(iK, 78);
    q = (kf * C[12]) * C[30] - (kr * C[26]) * C[26];
    om[12] -= q;
    om[30] -= q;
    om[26] += q;
    om[26] += q;
    kf = L.kf[79 * kLdsStride];
    kr = kf * ld_uniform(iK, 79);
    q = (kf * C[8]) * M - (kr * C[0]) * C[7];
    om[8] -= q;
    om[0] += q;
    om[7] += q;
    kf = L.kf[80 * kLdsStride];
    kr = kf * ld_uniform(iK, 80);
    q = (kf * C[14]) * C[30] - (kr * C[13]) * C[28];
    om[14] -= q;
    om[30] -= q;
    om[13] += q;
    om[28] += q;
    kf = L.kf[81 * kLdsStride];
    kr = kf * ld_uniform(iK, 81);
    q = (kf * C[4]) * C[4] - (kr * C[0]) * C[5];
    om[4] -= q;
    om[4] -= q;
    om[0] += q;
    om[5] += q;
    kf = L.kf[82 * kLdsStride];
    kr = kf * ld_uniform(iK, 82);
    q = (kf * C[9]) * C[20] - (kr * C[8]) * C[16];
    om[9] -= q;
    om[20] -= q;
    om[8] += q;
    om[16] += q;
    kf = L.kf[83 * kLdsStride];
    kr = kf * ld_uniform(iK, 83);
    q = (kf * C[6]) * C[17] - (kr * C[30]) * C[31];
    om[6] -= q;
    om[17] -= q;
    om[30] += q;
    om[31] += q;
    kf = L.kf[84 * kLdsStride];
    kr = kf * ld_uniform(iK, 84);
    q = (kf * C[5]) * C[16] - (kr * C[20]) * C[21];
    om[5] -= q;
    om[16] -= q;
    om[20] += q;
    om[21] += q;
    kf = L.kf[85 * kLdsStride];
    kr = kf * ld_uniform(iK, 85);
    q = (kf * C[12]) * C[14] - (kr * C[18]) * C[21];
    om[12] -= q;
    om[14] -= q;
    om[18] += q;
    om[21] += q;
    kf = L.kf[86 * kLdsStride];
    kr = kf * ld_uniform(iK, 86);
    q = (kf * C[14]) * C[30] - (kr * C[12]) * M;
    om[14] -= q;
    om[30] -= q;
    om[12] += q;
    kf = L.kf[87 * kLdsStride];
    kr = kf * ld_uniform(iK, 87);
    q = (kf * C[16]) * C[17] - (kr * C[12]) * C[15];
    om[16] -= q;
    om[17] -= q;
    om[12] += q;
    om[15] += q;
    kf = L.kf[88 * kLdsStride];
    kr = kf * ld_uniform(iK, 88);
    q = (kf * C[28]) * M - (kr * C[4]) * C[15];
    om[28] -= q;
    om[4] += q;
    om[15] += q;
    kf = L.kf[89 * kLdsStride];
    kr = kf * ld_uniform(iK, 89);
    q = (kf * C[2]) * C[10] - (kr * C[6]) * C[11];
    om[2] -= q;
    om[10] -= q;
    om[6] += q;
    om[11] += q;
    kf = L.kf[90 * kLdsStride];
    kr = kf * ld_uniform(iK, 90);
    q = (kf * C[31]) * M - (kr * C[0]) * C[20];
    om[31] -= q;
    om[0] += q;
    om[20] += q;
    kf = L.kf[91 * kLdsStride];
    kr = kf * ld_uniform(iK, 91);
    q = (kf * C[5]) * C[25] - (kr * C[9]) * C[14];
    om[5] -= q;
    om[25] -= q;
    om[9] += q;
    om[14] += q;
    kf = L.kf[92 * kLdsStride];
    kr = kf * ld_uniform(iK, 92);
    q = (kf * C[20]) * C[20] - (kr * C[6]) * C[14];
    om[20] -= q;
    om[20] -= q;
    om[6] += q;
    om[14] += q;
    kf = L.kf[93 * kLdsStride];
    kr = kf * ld_uniform(iK, 93);
    q = (kf * C[16]) * C[24] - (kr * C[3]) * C[18];
    om[16] -= q;
    om[24] -= q;
    om[3] += q;
    om[18] += q;
    kf = L.kf[94 * kLdsStride];
    kr = kf * ld_uniform(iK, 94);
    q = (kf * C[17]) * C[23] - (kr * C[8]) * C[25];
    om[17] -= q;
    om[23] -= q;
    om[8] += q;
    om[25] += q;
    kf = L.kf[95 * kLdsStride];
    kr = kf * ld_uniform(iK, 95);
    q = (kf * C[9]) * C[24] - (kr * C[4]) * C[12];
    om[9] -= q;
    om[24] -= q;
    om[4] += q;
    om[12] += q;
    kf = L.kf[96 * kLdsStride];
    kr = kf * ld_uniform(iK, 96);
    q = (kf * C[2]) * C[9] - (kr * C[1]) * C[17];
    om[2] -= q;
    om[9] -= q;
    om[1] += q;
    om[17] += q;
    kf = L.kf[97 * kLdsStride];
    kr = kf * ld_uniform(iK, 97);
    q = (kf * C[3]) * C[16] - (kr * C[20]) * C[20];
    om[3] -= q;
    om[16] -= q;
    om[20] += q;
    om[20] += q;
    kf = L.kf[98 * kLdsStride];
    kr = kf * ld_uniform(iK, 98);
    q = (kf * C[2]) * C[5] - (kr * C[0]) * C[24];
    om[2] -= q;
    om[5] -= q;
    om[0] += q;
    om[24] += q;
    kf = L.kf[99 * kLdsStride];
    kr = kf * ld_uniform(iK, 99);
    q = (kf * C[2]) * C[20] - (kr * C[11]) * C[15];
    om[2] -= q;
    om[20] -= q;
    om[11] += q;
    om[15] += q;
    kf = L.kf[100 * kLdsStride];
    kr = kf * ld_uniform(iK, 100);
    q = (kf * C[14]) * C[19] - (kr * C[2]) * C[9];
    om[14] -= q;
    om[19] -= q;
    om[2] += q;
    om[9] += q;
    kf = L.kf[101 * kLdsStride];
    kr = kf * ld_uniform(iK, 101);
    q = (kf * C[8]) * C[29] - (kr * C[3]) * C[18];
    om[8] -= q;
    om[29] -= q;
    om[3] += q;
    om[18] += q;
    kf = L.kf[102 * kLdsStride];
    kr = kf * ld_uniform(iK, 102);
    q = (kf * C[5]) * C[10] - (kr * C[6]) * C[22];
    om[5] -= q;
    om[10] -= q;
    om[6] += q;
    om[22] += q;
    kf = L.kf[103 * kLdsStride];
    kr = kf * ld_uniform(iK, 103);
    q = (kf * C[3]) * C[15] - (kr * C[1]) * C[4];
    om[3] -= q;
    om[15] -= q;
    om[1] += q;
    om[4] += q;
    kf = L.kf[104 * kLdsStride];
    kr = kf * ld_uniform(iK, 104);
    q = (kf * C[11]) * C[25] - (kr * C[2]) * C[26];
    om[11] -= q;
    om[25] -= q;
    om[2] += q;
    om[26] += q;
    kf = L.kf[105 * kLdsStride];
    kr = kf * ld_uniform(iK, 105);
    q = (kf * C[14]) * C[21] - (kr * C[24]) * C[28];
    om[14] -= q;
    om[21] -= q;
    om[24] += q;
    om[28] += q;
    kf = L.kf[106 * kLdsStride];
    kr = kf * ld_uniform(iK, 106);
    q = (kf * C[3]) * C[4] - (kr * C[0]) * C[14];
    om[3] -= q;
    om[4] -= q;
    om[0] += q;
    om[14] += q;
    kf = L.kf[107 * kLdsStride];
    kr = kf * ld_uniform(iK, 107);
    q = (kf * C[14]) * C[30] - (kr * C[2]) * C[27];
    om[14] -= q;
    om[30] -= q;
    om[2] += q;
    om[27] += q;
    kf = L.kf[108 * kLdsStride];
    kr = kf * ld_uniform(iK, 108);
    q = (kf * C[17]) * C[24] - (kr * C[5]) * C[18];
    om[17] -= q;
    om[24] -= q;
    om[5] += q;
    om[18] += q;
    kf = L.kf[109 * kLdsStride];
    kr = kf * ld_uniform(iK, 109);
    q = (kf * C[16]) * C[30] - (kr * C[10]) * C[25];
    om[16] -= q;
    om[30] -= q;
    om[10] += q;
    om[25] += q;
    kf = L.kf[110 * kLdsStride];
    kr = kf * ld_uniform(iK, 110);
    q = (kf * C[11]) * C[13] - (kr * C[10]) * C[29];
    om[11] -= q;
    om[13] -= q;
    om[10] += q;
    om[29] += q;
    kf = L.kf[111 * kLdsStride];
    kr = kf * ld_uniform(iK, 111);
    q = (kf * C[1]) * C[16] - (kr * C[6]) * C[20];
    om[1] -= q;
    om[16] -= q;
    om[6] += q;
    om[20] += q;
    kf = L.kf[112 * kLdsStride];
    kr = kf * ld_uniform(iK, 112);
    q = (kf * C[15]) * C[20] - (kr * C[1]) * C[31];
    om[15] -= q;
    om[20] -= q;
    om[1] += q;
    om[31] += q;
    kf = L.kf[113 * kLdsStride];
    kr = kf * ld_uniform(iK, 113);
    q = (kf * C[4]) * C[16] - (kr * C[17]) * M;
    om[4] -= q;
    om[16] -= q;
    om[17] += q;
    kf = L.kf[114 * kLdsStride];
    kr = kf * ld_uniform(iK, 114);
    q = (kf * C[30]) * M - (kr * C[1]) * C[16];
    om[30] -= q;
    om[1] += q;
    om[16] += q;
    kf = L.kf[115 * kLdsStride];
    kr = kf * ld_uniform(iK, 115);
    q = (kf * C[11]) * C[31] - (kr * C[1]) * C[24];
    om[11] -= q;
    om[31] -= q;
    om[1] += q;
    om[24] += q;
    kf = L.kf[116 * kLdsStride];
    kr = kf * ld_uniform(iK, 116);
    q = (kf * C[12]) * M - (kr * C[19]) * C[24];
    om[12] -= q;
    om[19] += q;
    om[24] += q;
    kf = L.kf[117 * kLdsStride];
    kr = kf * ld_uniform(iK, 117);
    q = (kf * C[21]) * C[27] - (kr * C[12]) * C[28];
    om[21] -= q;
    om[27] -= q;
    om[12] += q;
    om[28] += q;
    kf = L.kf[118 * kLdsStride];
    kr = kf * ld_uniform(iK, 118);
    q = (kf * C[1]) * C[26] - (kr * C[7]) * C[10];
    om[1] -= q;
    om[26] -= q;
    om[7] += q;
    om[10] += q;
    kf = L.kf[119 * kLdsStride];
    kr = kf * ld_uniform(iK, 119);
    q = (kf * C[1]) * C[17] - (kr * C[7]) * C[20];
    om[1] -= q;
    om[17] -= q;
    om[7] += q;
    om[20] += q;
    kf = L.kf[120 * kLdsStride];
    kr = kf * ld_uniform(iK, 120);
    q = (kf * C[0]) * C[27] - (kr * C[5]) * C[19];
    om[0] -= q;
    om[27] -= q;
    om[5] += q;
    om[19] += q;
    kf = L.kf[121 * kLdsStride];
    kr = kf * ld_uniform(iK, 121);
    q = (kf * C[4]) * C[26] - (kr * C[19]) * C[22];
    om[4] -= q;
    om[26] -= q;
    om[19] += q;
    om[22] += q;
    kf = L.kf[122 * kLdsStride];
    kr = kf * ld_uniform(iK, 122);
    q = (kf * C[12]) * C[14] - (kr * C[22]) * C[26];
    om[12] -= q;
    om[14] -= q;
    om[22] += q;
    om[26] += q;
    kf = L.kf[123 * kLdsStride];
    kr = kf * ld_uniform(iK, 123);
    q = (kf * C[22]) * C[25] - (kr * C[14]) * C[27];
    om[22] -= q;
    om[25] -= q;
    om[14] += q;
    om[27] += q;
    kf = L.kf[124 * kLdsStride];
    kr = kf * ld_uniform(iK, 124);
    q = (kf * C[4]) * C[26] - (kr * C[5]) * C[30];
    om[4] -= q;
    om[26] -= q;
    om[5] += q;
    om[30] += q;
    kf = L.kf[125 * kLdsStride];
    kr = kf * ld_uniform(iK, 125);
    q = (kf * C[17]) * C[20] - (kr * C[19]) * C[22];
    om[17] -= q;
    om[20] -= q;
    om[19] += q;
    om[22] += q;
    kf = L.kf[126 * kLdsStride];
    kr = kf * ld_uniform(iK, 126);
    q = (kf * C[10]) * C[17] - (kr * C[20]) * C[26];
    om[10] -= q;
    om[17] -= q;
    om[20] += q;
    om[26] += q;
    kf = L.kf[127 * kLdsStride];
    kr = kf * ld_uniform(iK, 127);
    q = (kf * C[25]) * C[28] - (kr * C[9]) * C[31];
    om[25] -= q;
    om[28] -= q;
    om[9] += q;
    om[31] += q;
    kf = L.kf[128 * kLdsStride];
    kr = kf * ld_uniform(iK, 128);
    q = (kf * C[7]) * C[28] - (kr * C[8]) * C[31];
    om[7] -= q;
    om[28] -= q;
    om[8] += q;
    om[31] += q;
    kf = L.kf[129 * kLdsStride];
    kr = kf * ld_uniform(iK, 129);
    q = (kf * C[3]) * C[9] - (kr * C[5]) * C[19];
    om[3] -= q;
    om[9] -= q;
    om[5] += q;
    om[19] += q;
    kf = L.kf[130 * kLdsStride];
    kr = kf * ld_uniform(iK, 130);
    q = (kf * C[16]) * C[22] - (kr * C[7]) * C[24];
    om[16] -= q;
    om[22] -= q;
    om[7] += q;
    om[24] += q;
    kf = L.kf[131 * kLdsStride];
    kr = kf * ld_uniform(iK, 131);
    q = (kf * C[10]) * C[28] - (kr * C[3]) * C[25];
    om[10] -= q;
    om[28] -= q;
    om[3] += q;
    om[25] += q;
    kf = L.kf[132 * kLdsStride];
    kr = kf * ld_uniform(iK, 132);
    q = (kf * C[22]) * C[31] - (kr * C[24]) * C[28];
    om[22] -= q;
    om[31] -= q;
    om[24] += q;
    om[28] += q;
#pragma unroll
    for (int k = 0; k < N; ++k) f[k] = (ld_uniform(W, k) * om[k]) * L.irho;
  }
};

// Group variant: 16 lanes per system (rk_group.hpp).
struct GNet {
  static constexpr int N = 32;
  static constexpr int NR = 133;
  static constexpr int kL = 16;
  static constexpr int kGroupLanes = 16;
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  // RKCK: three waves per SIMD, its loop fits 168 registers but for a few spills
  // outside the evaluations (53 species, 65536 systems, in one session: three waves
  // 636 ms, two 698)
  static constexpr int kWavesPerEuRkc = 2;
  static constexpr int kWavesPerEuRkck = 3;
  static constexpr int S = 2;
  static constexpr int R = 9;
  static constexpr int kMSlot = 8;   // first slot that may hold a [M] reaction
  static constexpr int kOffC = 0;
  static constexpr int kOffQ = 34;
  static constexpr int kSentinel = 144;
  static constexpr int kNegOff = 178;
  static constexpr int kOffRed = 180;
  static constexpr int kLdsPerSystem = 356;
  static constexpr int kTermLen = 40;
  static constexpr int kChunk = 4;
  using Params = const double*;
  static constexpr int kSp[32] = {
      20, 0, 4, 18, 11, 13, 26, 28, 3, 22, 21, 15, 12, 5, 10, 24,
      29, 14, 23, 16, 17, 25, 27, 8, 6, 19, 1, 9, 2, 7, 31, 30};
  static constexpr int16_t kRxOf[144] = {
      105, 22, -1, 47, -1, 29, 125, 9, 68, 72, -1, 55, -1, 129, 132, 34,
      115, 126, 112, 124, 60, 7, 28, 61, 97, 91, 130, 104, 118, 108, 92, 44,
      12, 48, 69, 62, 131, 106, 70, 81, 4, 109, 31, 63, 43, 11, 37, 103,
      6, 84, 20, 15, -1, 76, 100, 33, 99, 59, 14, 128, 13, 82, 27, -1,
      26, 40, 54, 39, 52, 87, 120, 36, 110, 94, 10, 127, 56, 8, 35, -1,
      85, 42, 5, 24, 30, 83, 57, 16, 107, 122, 111, 89, 119, 53, 96, 49,
      75, -1, 67, 51, 80, 23, 121, 38, 45, 19, 95, 102, 46, 98, 41, 0,
      117, 2, 93, 123, 32, 101, 78, 71, 65, 3, 64, 73, 21, 1, 50, 74,
      88, 114, 116, 58, 25, -1, 79, 17, -1, 77, 113, 86, 90, 18, 66, -1};
  // each lane's LDS offsets (in units of 2^kAddrShift bytes) in the wave's areas,
  // two to a word, contiguous and 16-byte aligned (read as whole vectors at every
  // evaluation): the rates' operands, the terms
  static constexpr int kAddrShift = 0;
  static constexpr int kOpWords = 20;
  static constexpr int kTmWords = 20;
  alignas(16) static constexpr uint32_t kOp[1280] = {
      11010160, 14680256, 16253016, 12582920, 12582984, 14680208, 11010128, 13631512, 14155968, 7340128, 7340128, 11010192, 15728672, 13107224, 14155944, 14680160,
      16777440, 7864352, 0, 0, 15204424, 10485904, 8912976, 13631648, 11010128, 15728752, 8388648, 11010208, 14680080, 7864432, 14155984, 13107296,
      0, 0, 14680160, 8913032, 16777456, 8388616, 0, 0, 0, 0, 10485880, 16252936, 3670048, 14680224, 16253120, 11534496,
      14155936, 15728808, 11010096, 9961584, 5767224, 6815776, 12583040, 9437208, 16777312, 12583064, 0, 0, 3670040, 4194320, 13631520, 15728680,
      15728824, 13107352, 11010176, 13107312, 6815784, 11534416, 8912928, 3670056, 14155784, 8912944, 13107376, 14155888, 13631512, 16777312, 0, 0,
      0, 0, 16253088, 3670040, 14680144, 13107224, 0, 0, 7340072, 11534368, 13631648, 6815808, 15728752, 14680168, 11010128, 9437304,
      16777392, 7340056, 0, 0, 7864392, 14680216, 13631512, 14680168, 2097176, 7340032, 11534392, 8913008, 8913024, 7864416, 8912944, 16253168,
      14680144, 9961584, 15204416, 9437208, 0, 0, 0, 0, 10485896, 11534488, 4718600, 13107320, 13631512, 5767240, 9961584, 4718608,
      14155776, 9961512, 6291496, 14155952, 13631520, 11534488, 15728736, 13631696, 16777280, 3670016, 0, 0, 11010112, 4718632, 10485880, 3145760,
      2097184, 2621440, 13107312, 12583096, 11534360, 7340144, 10485816, 14680144, 13631496, 8388736, 12058736, 8913016, 1048592, 16777304, 0, 0,
      15204424, 11010152, 8388632, 10485920, 13107272, 14155960, 10485776, 7864408, 6815832, 15204432, 15728752, 14155792, 15728672, 8912904, 16253152, 4194336,
      0, 0, 0, 0, 16252952, 14680080, 13107240, 7340104, 15728768, 13107280, 11534456, 10485800, 12058760, 13107264, 7340128, 13631664,
      11010176, 10485896, 12058800, 14155808, 16777344, 5242880, 0, 0, 0, 0, 11534464, 12582968, 16253112, 14680216, 11534344, 11010064,
      7340120, 12582928, 8388616, 10485808, 12582984, 6291488, 11010168, 4194328, 8388640, 16777352, 0, 0, 15728816, 16253072, 13107288, 13631504,
      13107400, 15728712, 14680120, 16252992, 14680264, 16253000, 5242896, 5767216, 5242920, 11534384, 13631552, 13107336, 15728752, 16777312, 0, 0,
      0, 0, 13631496, 5242936, 12583040, 11534416, 8912984, 6815784, 14155800, 10485896, 8912904, 10485816, 9961616, 6291504, 11010208, 8912920,
      16777464, 10485760, 0, 0, 4718616, 9961512, 12583048, 9437224, 8388680, 13107256, 10485832, 8388672, 14680272, 13107368, 12058736, 10485824,
      2621456, 12582912, 15728760, 3670064, 16777432, 11010096, 0, 0, 16253104, 14680256, 10485920, 7340080, 13631616, 6291504, 13631488, 4718608,
      13631504, 16253032, 4718608, 8912904, 14680168, 12583064, 11534488, 13107312, 13107216, 16777424, 0, 0, 9437232, 6815800, 16253008, 10485888,
      7864344, 2097160, 0, 0, 0, 0, 8388640, 16253088, 7864384, 12058656, 11010056, 8388640, 0, 0, 0, 0,
      197659536, 201329632, 202902392, 199232296, 199232360, 201329584, 197659504, 200280888, 200805344, 193989504, 193989504, 197659568, 202378048, 199756600, 200805320, 201329536,
      203426816, 194513728, 0, 0, 201853800, 197135280, 195562352, 200281024, 197659504, 202378128, 195038024, 197659584, 201329456, 194513808, 200805360, 199756672,
      186649376, 186649376, 201329536, 195562408, 203426832, 195037992, 0, 0, 186649376, 186649376, 197135256, 202902312, 190319424, 201329600, 202902496, 198183872,
      200805312, 202378184, 197659472, 196610960, 192416600, 193465152, 199232416, 196086584, 203426688, 199232440, 0, 0, 190319416, 190843696, 200280896, 202378056,
      202378200, 199756728, 197659552, 199756688, 193465160, 198183792, 195562304, 190319432, 200805160, 195562320, 199756752, 200805264, 200280888, 203426688, 0, 0,
      186649376, 186649376, 202902464, 190319416, 201329520, 199756600, 186649376, 186649376, 193989448, 198183744, 200281024, 193465184, 202378128, 201329544, 197659504, 196086680,
      203426768, 193989432, 0, 0, 194513768, 201329592, 200280888, 201329544, 188746552, 193989408, 198183768, 195562384, 195562400, 194513792, 195562320, 202902544,
      201329520, 196610960, 201853792, 196086584, 186649376, 186649376, 0, 0, 197135272, 198183864, 191367976, 199756696, 200280888, 192416616, 196610960, 191367984,
      200805152, 196610888, 192940872, 200805328, 200280896, 198183864, 202378112, 200281072, 203426656, 190319392, 0, 0, 197659488, 191368008, 197135256, 189795136,
      188746560, 189270816, 199756688, 199232472, 198183736, 193989520, 197135192, 201329520, 200280872, 195038112, 198708112, 195562392, 187697968, 203426680, 0, 0,
      201853800, 197659528, 195038008, 197135296, 199756648, 200805336, 197135152, 194513784, 193465208, 201853808, 202378128, 200805168, 202378048, 195562280, 202902528, 190843712,
      186649376, 186649376, 0, 0, 202902328, 201329456, 199756616, 193989480, 202378144, 199756656, 198183832, 197135176, 198708136, 199756640, 193989504, 200281040,
      197659552, 197135272, 198708176, 200805184, 203426720, 191892256, 0, 0, 186649376, 186649376, 198183840, 199232344, 202902488, 201329592, 198183720, 197659440,
      193989496, 199232304, 195037992, 197135184, 199232360, 192940864, 197659544, 190843704, 195038016, 203426728, 0, 0, 202378192, 202902448, 199756664, 200280880,
      199756776, 202378088, 201329496, 202902368, 201329640, 202902376, 191892272, 192416592, 191892296, 198183760, 200280928, 199756712, 202378128, 203426688, 0, 0,
      186649376, 186649376, 200280872, 191892312, 199232416, 198183792, 195562360, 193465160, 200805176, 197135272, 195562280, 197135192, 196610992, 192940880, 197659584, 195562296,
      203426840, 197135136, 0, 0, 191367992, 196610888, 199232424, 196086600, 195038056, 199756632, 197135208, 195038048, 201329648, 199756744, 198708112, 197135200,
      189270832, 199232288, 202378136, 190319440, 203426808, 197659472, 0, 0, 202902480, 201329632, 197135296, 193989456, 200280992, 192940880, 200280864, 191367984,
      200280880, 202902408, 191367984, 195562280, 201329544, 199232440, 198183864, 199756688, 199756592, 203426800, 0, 0, 196086608, 193465176, 202902384, 197135264,
      194513720, 188746536, 186649376, 186649376, 186649376, 186649376, 195038016, 202902464, 194513760, 198708032, 197659432, 195038016, 186649376, 186649376, 0, 0,
      384308912, 387979008, 389551768, 385881672, 385881736, 387978960, 384308880, 386930264, 387454720, 380638880, 380638880, 384308944, 389027424, 386405976, 387454696, 387978912,
      390076192, 381163104, 0, 0, 388503176, 383784656, 382211728, 386930400, 384308880, 389027504, 381687400, 384308960, 387978832, 381163184, 387454736, 386406048,
      373298752, 373298752, 387978912, 382211784, 390076208, 381687368, 0, 0, 373298752, 373298752, 383784632, 389551688, 376968800, 387978976, 389551872, 384833248,
      387454688, 389027560, 384308848, 383260336, 379065976, 380114528, 385881792, 382735960, 390076064, 385881816, 0, 0, 376968792, 377493072, 386930272, 389027432,
      389027576, 386406104, 384308928, 386406064, 380114536, 384833168, 382211680, 376968808, 387454536, 382211696, 386406128, 387454640, 386930264, 390076064, 0, 0,
      373298752, 373298752, 389551840, 376968792, 387978896, 386405976, 373298752, 373298752, 380638824, 384833120, 386930400, 380114560, 389027504, 387978920, 384308880, 382736056,
      390076144, 380638808, 0, 0, 381163144, 387978968, 386930264, 387978920, 375395928, 380638784, 384833144, 382211760, 382211776, 381163168, 382211696, 389551920,
      387978896, 383260336, 388503168, 382735960, 373298752, 373298752, 0, 0, 383784648, 384833240, 378017352, 386406072, 386930264, 379065992, 383260336, 378017360,
      387454528, 383260264, 379590248, 387454704, 386930272, 384833240, 389027488, 386930448, 390076032, 376968768, 0, 0, 384308864, 378017384, 383784632, 376444512,
      375395936, 375920192, 386406064, 385881848, 384833112, 380638896, 383784568, 387978896, 386930248, 381687488, 385357488, 382211768, 374347344, 390076056, 0, 0,
      388503176, 384308904, 381687384, 383784672, 386406024, 387454712, 383784528, 381163160, 380114584, 388503184, 389027504, 387454544, 389027424, 382211656, 389551904, 377493088,
      373298752, 373298752, 0, 0, 389551704, 387978832, 386405992, 380638856, 389027520, 386406032, 384833208, 383784552, 385357512, 386406016, 380638880, 386930416,
      384308928, 383784648, 385357552, 387454560, 390076096, 378541632, 0, 0, 373298752, 373298752, 384833216, 385881720, 389551864, 387978968, 384833096, 384308816,
      380638872, 385881680, 381687368, 383784560, 385881736, 379590240, 384308920, 377493080, 381687392, 390076104, 0, 0, 389027568, 389551824, 386406040, 386930256,
      386406152, 389027464, 387978872, 389551744, 387979016, 389551752, 378541648, 379065968, 378541672, 384833136, 386930304, 386406088, 389027504, 390076064, 0, 0,
      373298752, 373298752, 386930248, 378541688, 385881792, 384833168, 382211736, 380114536, 387454552, 383784648, 382211656, 383784568, 383260368, 379590256, 384308960, 382211672,
      390076216, 383784512, 0, 0, 378017368, 383260264, 385881800, 382735976, 381687432, 386406008, 383784584, 381687424, 387979024, 386406120, 385357488, 383784576,
      375920208, 385881664, 389027512, 376968816, 390076184, 384308848, 0, 0, 389551856, 387979008, 383784672, 380638832, 386930368, 379590256, 386930240, 378017360,
      386930256, 389551784, 378017360, 382211656, 387978920, 385881816, 384833240, 386406064, 386405968, 390076176, 0, 0, 382735984, 380114552, 389551760, 383784640,
      381163096, 375395912, 373298752, 373298752, 373298752, 373298752, 381687392, 389551840, 381163136, 385357408, 384308808, 381687392, 373298752, 373298752, 0, 0,
      570958288, 574628384, 576201144, 572531048, 572531112, 574628336, 570958256, 573579640, 574104096, 567288256, 567288256, 570958320, 575676800, 573055352, 574104072, 574628288,
      576725568, 567812480, 0, 0, 575152552, 570434032, 568861104, 573579776, 570958256, 575676880, 568336776, 570958336, 574628208, 567812560, 574104112, 573055424,
      559948128, 559948128, 574628288, 568861160, 576725584, 568336744, 0, 0, 559948128, 559948128, 570434008, 576201064, 563618176, 574628352, 576201248, 571482624,
      574104064, 575676936, 570958224, 569909712, 565715352, 566763904, 572531168, 569385336, 576725440, 572531192, 0, 0, 563618168, 564142448, 573579648, 575676808,
      575676952, 573055480, 570958304, 573055440, 566763912, 571482544, 568861056, 563618184, 574103912, 568861072, 573055504, 574104016, 573579640, 576725440, 0, 0,
      559948128, 559948128, 576201216, 563618168, 574628272, 573055352, 559948128, 559948128, 567288200, 571482496, 573579776, 566763936, 575676880, 574628296, 570958256, 569385432,
      576725520, 567288184, 0, 0, 567812520, 574628344, 573579640, 574628296, 562045304, 567288160, 571482520, 568861136, 568861152, 567812544, 568861072, 576201296,
      574628272, 569909712, 575152544, 569385336, 559948128, 559948128, 0, 0, 570434024, 571482616, 564666728, 573055448, 573579640, 565715368, 569909712, 564666736,
      574103904, 569909640, 566239624, 574104080, 573579648, 571482616, 575676864, 573579824, 576725408, 563618144, 0, 0, 570958240, 564666760, 570434008, 563093888,
      562045312, 562569568, 573055440, 572531224, 571482488, 567288272, 570433944, 574628272, 573579624, 568336864, 572006864, 568861144, 560996720, 576725432, 0, 0,
      575152552, 570958280, 568336760, 570434048, 573055400, 574104088, 570433904, 567812536, 566763960, 575152560, 575676880, 574103920, 575676800, 568861032, 576201280, 564142464,
      559948128, 559948128, 0, 0, 576201080, 574628208, 573055368, 567288232, 575676896, 573055408, 571482584, 570433928, 572006888, 573055392, 567288256, 573579792,
      570958304, 570434024, 572006928, 574103936, 576725472, 565191008, 0, 0, 559948128, 559948128, 571482592, 572531096, 576201240, 574628344, 571482472, 570958192,
      567288248, 572531056, 568336744, 570433936, 572531112, 566239616, 570958296, 564142456, 568336768, 576725480, 0, 0, 575676944, 576201200, 573055416, 573579632,
      573055528, 575676840, 574628248, 576201120, 574628392, 576201128, 565191024, 565715344, 565191048, 571482512, 573579680, 573055464, 575676880, 576725440, 0, 0,
      559948128, 559948128, 573579624, 565191064, 572531168, 571482544, 568861112, 566763912, 574103928, 570434024, 568861032, 570433944, 569909744, 566239632, 570958336, 568861048,
      576725592, 570433888, 0, 0, 564666744, 569909640, 572531176, 569385352, 568336808, 573055384, 570433960, 568336800, 574628400, 573055496, 572006864, 570433952,
      562569584, 572531040, 575676888, 563618192, 576725560, 570958224, 0, 0, 576201232, 574628384, 570434048, 567288208, 573579744, 566239632, 573579616, 564666736,
      573579632, 576201160, 564666736, 568861032, 574628296, 572531192, 571482616, 573055440, 573055344, 576725552, 0, 0, 569385360, 566763928, 576201136, 570434016,
      567812472, 562045288, 559948128, 559948128, 559948128, 559948128, 568336768, 576201216, 567812512, 572006784, 570958184, 568336768, 559948128, 559948128, 0, 0};
  alignas(16) static constexpr uint32_t kTm[1280] = {
      72878424, 176161440, 155189528, 67633672, 145753080, 47711088, 123209536, 143131168, 91226776, 126879632, 30409168, 65013856, 66062128, 26740432, 115345064, 55577160,
      93324688, 93324688, 93324688, 93324688, 89655440, 38274368, 74974576, 147849784, 149947296, 70779560, 51381552, 55052376, 51905352, 83886616, 159910080, 45615704,
      153094592, 30935800, 139461120, 37226144, 157813088, 93324456, 93324688, 93324688, 81265800, 165677368, 53479832, 80740808, 128975904, 161481992, 131598296, 73401616,
      130548360, 164629232, 93325112, 93324688, 174589064, 133169744, 159908552, 173541304, 93325544, 93324688, 93324688, 93324688, 18350608, 119014576, 23595520, 77595536,
      33031352, 93324688, 137889800, 135268840, 71828552, 34080768, 84412824, 49810152, 147327016, 123734576, 158337000, 85461744, 93325168, 93324688, 93324688, 93324688,
      142608624, 162530632, 65536576, 125305552, 119539936, 93324688, 77071512, 72878208, 154666224, 69731408, 80216944, 45614312, 147327304, 67111144, 90179464, 114297216,
      93325096, 93324688, 93324688, 93324688, 49283512, 25691056, 146277248, 69208592, 70254928, 93325536, 58197984, 44565112, 139985344, 83887000, 133693992, 185599992,
      68158696, 56100712, 39323512, 150473272, 93323824, 93324688, 93324688, 93324688, 122159760, 143657224, 152045888, 165152784, 179833128, 131073408, 79694456, 31982784,
      164628352, 121111512, 93323672, 93324688, 38798552, 144706312, 163055912, 150997168, 63964096, 147851808, 93324456, 93324688, 28838440, 34605320, 164103112, 39846200,
      168822952, 35654240, 70254936, 17828512, 150471824, 130025592, 93323648, 93324688, 114821656, 19399600, 81789944, 175637712, 49810128, 172491608, 93324008, 93324688,
      122159760, 87033072, 112724184, 179833088, 81789360, 115869648, 77595664, 79169376, 130549784, 36701960, 154141944, 119014776, 74449536, 29885480, 65538376, 73925120,
      93324256, 93324688, 93324688, 93324688, 141560424, 180355744, 52955352, 177209968, 116917040, 141034432, 73926728, 64488512, 20974136, 118490992, 70779808, 39846200,
      167773312, 36178576, 85985360, 71304000, 24641856, 93324688, 93324688, 93324688, 136317232, 114819960, 137888480, 166200696, 171969152, 52430760, 22022768, 43518616,
      111149968, 93325856, 122685552, 72354264, 177736120, 42468352, 27265392, 26215704, 159385472, 93324688, 93324688, 93324688, 176687640, 113770944, 51905712, 123209832,
      80218736, 84935480, 135791312, 93325104, 21497824, 127928328, 50333352, 113772368, 115343976, 143131200, 166724056, 46139792, 117965672, 93324688, 93324688, 93324688,
      51382824, 60293760, 156238960, 173016360, 90704160, 73401144, 76548784, 93325672, 48235360, 181930712, 152044288, 19400872, 22547216, 160434552, 140511752, 31982272,
      93324240, 93324688, 93324688, 93324688, 49283400, 146277288, 156240064, 38273752, 124258344, 167250440, 54526456, 24641960, 41420024, 61344088, 112722312, 162529712,
      138938288, 32507200, 142083056, 93323744, 93324688, 93324688, 93324688, 93324688, 63440928, 171968968, 40895272, 128452504, 158860632, 39324152, 32506704, 130025256,
      133171248, 127402880, 23593992, 174065472, 62392040, 27265792, 57149216, 118489832, 93324688, 93324688, 93324688, 93324688, 127927136, 144705584, 75498184, 170919936,
      74975728, 126353680, 85983632, 25166304, 165677704, 52429336, 129500920, 161481320, 163580496, 184026040, 132647264, 27789992, 93324688, 93324688, 93324688, 93324688,
      259527800, 362810816, 341838904, 254283048, 332402456, 234360464, 309858912, 329780544, 277876152, 313529008, 217058544, 251663232, 252711504, 213389808, 301994440, 242226536,
      279974064, 279974064, 279974064, 279974064, 276304816, 224923744, 261623952, 334499160, 336596672, 257428936, 238030928, 241701752, 238554728, 270535992, 346559456, 232265080,
      339743968, 217585176, 326110496, 223875520, 344462464, 279973832, 279974064, 279974064, 267915176, 352326744, 240129208, 267390184, 315625280, 348131368, 318247672, 260050992,
      317197736, 351278608, 279974488, 279974064, 361238440, 319819120, 346557928, 360190680, 279974920, 279974064, 279974064, 279974064, 204999984, 305663952, 210244896, 264244912,
      219680728, 279974064, 324539176, 321918216, 258477928, 220730144, 271062200, 236459528, 333976392, 310383952, 344986376, 272111120, 279974544, 279974064, 279974064, 279974064,
      329258000, 349180008, 252185952, 311954928, 306189312, 279974064, 263720888, 259527584, 341315600, 256380784, 266866320, 232263688, 333976680, 253760520, 276828840, 300946592,
      279974472, 279974064, 279974064, 279974064, 235932888, 212340432, 332926624, 255857968, 256904304, 279974912, 244847360, 231214488, 326634720, 270536376, 320343368, 372249368,
      254808072, 242750088, 225972888, 337122648, 279973200, 279974064, 279974064, 279974064, 308809136, 330306600, 338695264, 351802160, 366482504, 317722784, 266343832, 218632160,
      351277728, 307760888, 279973048, 279974064, 225447928, 331355688, 349705288, 337646544, 250613472, 334501184, 279973832, 279974064, 215487816, 221254696, 350752488, 226495576,
      355472328, 222303616, 256904312, 204477888, 337121200, 316674968, 279973024, 279974064, 301471032, 206048976, 268439320, 362287088, 236459504, 359140984, 279973384, 279974064,
      308809136, 273682448, 299373560, 366482464, 268438736, 302519024, 264245040, 265818752, 317199160, 223351336, 340791320, 305664152, 261098912, 216534856, 252187752, 260574496,
      279973632, 279974064, 279974064, 279974064, 328209800, 367005120, 239604728, 363859344, 303566416, 327683808, 260576104, 251137888, 207623512, 305140368, 257429184, 226495576,
      354422688, 222827952, 272634736, 257953376, 211291232, 279974064, 279974064, 279974064, 322966608, 301469336, 324537856, 352850072, 358618528, 239080136, 208672144, 230167992,
      297799344, 279975232, 309334928, 259003640, 364385496, 229117728, 213914768, 212865080, 346034848, 279974064, 279974064, 279974064, 363337016, 300420320, 238555088, 309859208,
      266868112, 271584856, 322440688, 279974480, 208147200, 314577704, 236982728, 300421744, 301993352, 329780576, 353373432, 232789168, 304615048, 279974064, 279974064, 279974064,
      238032200, 246943136, 342888336, 359665736, 277353536, 260050520, 263198160, 279975048, 234884736, 368580088, 338693664, 206050248, 209196592, 347083928, 327161128, 218631648,
      279973616, 279974064, 279974064, 279974064, 235932776, 332926664, 342889440, 224923128, 310907720, 353899816, 241175832, 211291336, 228069400, 247993464, 299371688, 349179088,
      325587664, 219156576, 328732432, 279973120, 279974064, 279974064, 279974064, 279974064, 250090304, 358618344, 227544648, 315101880, 345510008, 225973528, 219156080, 316674632,
      319820624, 314052256, 210243368, 360714848, 249041416, 213915168, 243798592, 305139208, 279974064, 279974064, 279974064, 279974064, 314576512, 331354960, 262147560, 357569312,
      261625104, 313003056, 272633008, 211815680, 352327080, 239078712, 316150296, 348130696, 350229872, 370675416, 319296640, 214439368, 279974064, 279974064, 279974064, 279974064,
      446177176, 549460192, 528488280, 440932424, 519051832, 421009840, 496508288, 516429920, 464525528, 500178384, 403707920, 438312608, 439360880, 400039184, 488643816, 428875912,
      466623440, 466623440, 466623440, 466623440, 462954192, 411573120, 448273328, 521148536, 523246048, 444078312, 424680304, 428351128, 425204104, 457185368, 533208832, 418914456,
      526393344, 404234552, 512759872, 410524896, 531111840, 466623208, 466623440, 466623440, 454564552, 538976120, 426778584, 454039560, 502274656, 534780744, 504897048, 446700368,
      503847112, 537927984, 466623864, 466623440, 547887816, 506468496, 533207304, 546840056, 466624296, 466623440, 466623440, 466623440, 391649360, 492313328, 396894272, 450894288,
      406330104, 466623440, 511188552, 508567592, 445127304, 407379520, 457711576, 423108904, 520625768, 497033328, 531635752, 458760496, 466623920, 466623440, 466623440, 466623440,
      515907376, 535829384, 438835328, 498604304, 492838688, 466623440, 450370264, 446176960, 527964976, 443030160, 453515696, 418913064, 520626056, 440409896, 463478216, 487595968,
      466623848, 466623440, 466623440, 466623440, 422582264, 398989808, 519576000, 442507344, 443553680, 466624288, 431496736, 417863864, 513284096, 457185752, 506992744, 558898744,
      441457448, 429399464, 412622264, 523772024, 466622576, 466623440, 466623440, 466623440, 495458512, 516955976, 525344640, 538451536, 553131880, 504372160, 452993208, 405281536,
      537927104, 494410264, 466622424, 466623440, 412097304, 518005064, 536354664, 524295920, 437262848, 521150560, 466623208, 466623440, 402137192, 407904072, 537401864, 413144952,
      542121704, 408952992, 443553688, 391127264, 523770576, 503324344, 466622400, 466623440, 488120408, 392698352, 455088696, 548936464, 423108880, 545790360, 466622760, 466623440,
      495458512, 460331824, 486022936, 553131840, 455088112, 489168400, 450894416, 452468128, 503848536, 410000712, 527440696, 492313528, 447748288, 403184232, 438837128, 447223872,
      466623008, 466623440, 466623440, 466623440, 514859176, 553654496, 426254104, 550508720, 490215792, 514333184, 447225480, 437787264, 394272888, 491789744, 444078560, 413144952,
      541072064, 409477328, 459284112, 444602752, 397940608, 466623440, 466623440, 466623440, 509615984, 488118712, 511187232, 539499448, 545267904, 425729512, 395321520, 416817368,
      484448720, 466624608, 495984304, 445653016, 551034872, 415767104, 400564144, 399514456, 532684224, 466623440, 466623440, 466623440, 549986392, 487069696, 425204464, 496508584,
      453517488, 458234232, 509090064, 466623856, 394796576, 501227080, 423632104, 487071120, 488642728, 516429952, 540022808, 419438544, 491264424, 466623440, 466623440, 466623440,
      424681576, 433592512, 529537712, 546315112, 464002912, 446699896, 449847536, 466624424, 421534112, 555229464, 525343040, 392699624, 395845968, 533733304, 513810504, 405281024,
      466622992, 466623440, 466623440, 466623440, 422582152, 519576040, 529538816, 411572504, 497557096, 540549192, 427825208, 397940712, 414718776, 434642840, 486021064, 535828464,
      512237040, 405805952, 515381808, 466622496, 466623440, 466623440, 466623440, 466623440, 436739680, 545267720, 414194024, 501751256, 532159384, 412622904, 405805456, 503324008,
      506470000, 500701632, 396892744, 547364224, 435690792, 400564544, 430447968, 491788584, 466623440, 466623440, 466623440, 466623440, 501225888, 518004336, 448796936, 544218688,
      448274480, 499652432, 459282384, 398465056, 538976456, 425728088, 502799672, 534780072, 536879248, 557324792, 505946016, 401088744, 466623440, 466623440, 466623440, 466623440,
      632826552, 736109568, 715137656, 627581800, 705701208, 607659216, 683157664, 703079296, 651174904, 686827760, 590357296, 624961984, 626010256, 586688560, 675293192, 615525288,
      653272816, 653272816, 653272816, 653272816, 649603568, 598222496, 634922704, 707797912, 709895424, 630727688, 611329680, 615000504, 611853480, 643834744, 719858208, 605563832,
      713042720, 590883928, 699409248, 597174272, 717761216, 653272584, 653272816, 653272816, 641213928, 725625496, 613427960, 640688936, 688924032, 721430120, 691546424, 633349744,
      690496488, 724577360, 653273240, 653272816, 734537192, 693117872, 719856680, 733489432, 653273672, 653272816, 653272816, 653272816, 578298736, 678962704, 583543648, 637543664,
      592979480, 653272816, 697837928, 695216968, 631776680, 594028896, 644360952, 609758280, 707275144, 683682704, 718285128, 645409872, 653273296, 653272816, 653272816, 653272816,
      702556752, 722478760, 625484704, 685253680, 679488064, 653272816, 637019640, 632826336, 714614352, 629679536, 640165072, 605562440, 707275432, 627059272, 650127592, 674245344,
      653273224, 653272816, 653272816, 653272816, 609231640, 585639184, 706225376, 629156720, 630203056, 653273664, 618146112, 604513240, 699933472, 643835128, 693642120, 745548120,
      628106824, 616048840, 599271640, 710421400, 653271952, 653272816, 653272816, 653272816, 682107888, 703605352, 711994016, 725100912, 739781256, 691021536, 639642584, 591930912,
      724576480, 681059640, 653271800, 653272816, 598746680, 704654440, 723004040, 710945296, 623912224, 707799936, 653272584, 653272816, 588786568, 594553448, 724051240, 599794328,
      728771080, 595602368, 630203064, 577776640, 710419952, 689973720, 653271776, 653272816, 674769784, 579347728, 641738072, 735585840, 609758256, 732439736, 653272136, 653272816,
      682107888, 646981200, 672672312, 739781216, 641737488, 675817776, 637543792, 639117504, 690497912, 596650088, 714090072, 678962904, 634397664, 589833608, 625486504, 633873248,
      653272384, 653272816, 653272816, 653272816, 701508552, 740303872, 612903480, 737158096, 676865168, 700982560, 633874856, 624436640, 580922264, 678439120, 630727936, 599794328,
      727721440, 596126704, 645933488, 631252128, 584589984, 653272816, 653272816, 653272816, 696265360, 674768088, 697836608, 726148824, 731917280, 612378888, 581970896, 603466744,
      671098096, 653273984, 682633680, 632302392, 737684248, 602416480, 587213520, 586163832, 719333600, 653272816, 653272816, 653272816, 736635768, 673719072, 611853840, 683157960,
      640166864, 644883608, 695739440, 653273232, 581445952, 687876456, 610281480, 673720496, 675292104, 703079328, 726672184, 606087920, 677913800, 653272816, 653272816, 653272816,
      611330952, 620241888, 716187088, 732964488, 650652288, 633349272, 636496912, 653273800, 608183488, 741878840, 711992416, 579349000, 582495344, 720382680, 700459880, 591930400,
      653272368, 653272816, 653272816, 653272816, 609231528, 706225416, 716188192, 598221880, 684206472, 727198568, 614474584, 584590088, 601368152, 621292216, 672670440, 722477840,
      698886416, 592455328, 702031184, 653271872, 653272816, 653272816, 653272816, 653272816, 623389056, 731917096, 600843400, 688400632, 718808760, 599272280, 592454832, 689973384,
      693119376, 687351008, 583542120, 734013600, 622340168, 587213920, 617097344, 678437960, 653272816, 653272816, 653272816, 653272816, 687875264, 704653712, 635446312, 730868064,
      634923856, 686301808, 645931760, 585114432, 725625832, 612377464, 689449048, 721429448, 723528624, 743974168, 692595392, 587738120, 653272816, 653272816, 653272816, 653272816};
  static constexpr int kBnd[16] = {
      7, 2, 6, 3, 3, 3, 6, 6, 5, 5, 5, 4, 4, 4, 4, 4};
  // chunks at whose end some lane moves its accumulator to slot 0 (bit c)
  static constexpr uint64_t kSwitchChunks = 126ull;
  struct Lane {
    double kf[R], kr[R];
    double W[S], iW[S];
    double rho, irho;
    int bnd;   // chunks of the slot-0 list
  };
  // The forward rate constants of a lane's positions into the group's rate
  // area; once per system, out of line (the exponentials' temporaries do not
  // count against the registers of the evaluation loop).
  __device__ __attribute__((noinline)) static void rates(Params p, double T, double* lds, int r) {
    const double lnT = crm::cr_log(T);
    double* const Q = lds + kOffQ;
#pragma nounroll
    for (int m = 0; m < R; ++m) {
      const int j = kRxOf[m * kL + r];
      if (j >= 0) Q[m * kL + r] = crm::cr_exp(p[j] + p[NR + j] * lnT - p[2 * NR + j] / T);
    }
  }
  __device__ static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                              int64_t n, const Grp<GNet>& x) {
    const double T = g[i];
    const double rho = g[n + i];
    double* const Q = x.lds + kOffQ;
    rates(p, T, x.lds, x.r);
#pragma unroll
    for (int m = 0; m < R; ++m) {
      const int j = kRxOf[m * kL + x.r];
      L.kf[m] = j >= 0 ? Q[m * kL + x.r] : 0.0;
      L.kr[m] = j >= 0 ? L.kf[m] * p[3 * NR + j] : 0.0;
    }
#pragma unroll
    for (int m = 0; m < S; ++m) {
      const int k = x.sp[m];
      L.W[m] = k >= 0 ? p[4 * NR + k] : 0.0;
      L.iW[m] = k >= 0 ? p[4 * NR + N + k] : 0.0;
    }
    L.rho = rho;
    L.irho = 1.0 / rho;
    L.bnd = kBnd[x.r];
    if (x.r == 0) Q[kSentinel] = 0.0;
  }
};

// Wide variant: 32 lanes per system, one species per lane (rk_group.hpp).
struct WNet {
  static constexpr bool kWide = true;
  // largest batches it runs, in systems per SIMD (rk_group.hpp group_rhs_wide)
  static constexpr int kMaxRkck = 48;
  static constexpr int kMaxRkc = 6;
  static constexpr int N = 32;
  static constexpr int NR = 133;
  static constexpr int kL = 32;
  static constexpr int kGroupLanes = 32;
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  static constexpr int kWavesPerEuRkc = 2;
  static constexpr int kWavesPerEuRkck = 2;
  static constexpr int S = 1;
  static constexpr int R = 5;
  static constexpr int kMSlot = 4;   // first slot that may hold a [M] reaction
  static constexpr int kOffC = 0;
  static constexpr int kOffQ = 34;
  static constexpr int kOffZero = 194;
  static constexpr int kNegOff = 256;
  static constexpr int kOffRed = 196;
  static constexpr int kLdsPerSystem = 450;
  static constexpr int kTermLen = 28;
  using Params = const double*;
  static constexpr int kSp[32] = {
      0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15,
      16, 17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31};
  static constexpr int16_t kRxOf[160] = {
      83, 73, 82, 5, 120, 52, 67, 24, -1, 65, 36, 63, 2, -1, 42, 91,
      128, 122, 32, 80, 6, 121, 110, 22, 81, 45, 31, 41, 118, 100, 64, 115,
      -1, 51, 26, 96, 27, -1, 35, 111, 127, 55, 106, 126, 34, -1, 1, 85,
      132, 29, 103, 3, 28, 107, 4, 15, 131, 93, 0, 108, 37, 33, 104, 61,
      19, 94, 71, 117, 8, 40, 97, 56, 98, 11, 101, 95, 119, 48, 76, 102,
      14, 57, 74, 123, 70, 21, 46, 84, 30, 105, 69, 124, 62, 54, 49, 20,
      16, 9, 53, -1, 44, 87, 13, 92, 59, 130, 47, 38, 60, 12, 78, 39,
      -1, 75, 43, 50, 125, 99, 68, -1, 23, 89, 109, 129, 112, 72, 10, 7,
      -1, -1, -1, -1, 113, -1, 86, -1, -1, 90, 114, 25, -1, 88, 18, 17,
      -1, -1, 66, -1, -1, -1, -1, -1, 58, -1, 77, -1, 79, -1, 116, -1};
  // LDS byte offsets within the system's area: each lane's rate operands
  // (R x 4), and the signed rates of its species in reaction order
  alignas(16) static constexpr uint16_t kOp[640] = {
      48, 136, 240, 248, 0, 0, 0, 0, 128, 168, 136, 160, 56, 160, 80, 224,
      0, 0, 0, 0, 64, 208, 136, 200, 8, 216, 48, 136, 136, 184, 64, 200,
      64, 168, 40, 72, 0, 0, 0, 0, 72, 160, 64, 128, 192, 216, 96, 112,
      112, 184, 120, 136, 112, 184, 64, 160, 0, 0, 0, 0, 48, 168, 112, 152,
      16, 72, 8, 136, 168, 216, 96, 224, 0, 0, 0, 0, 0, 0, 0, 0,
      0, 216, 40, 152, 0, 208, 16, 72, 208, 224, 168, 200, 80, 248, 128, 160,
      32, 128, 136, 256, 40, 112, 32, 176, 0, 0, 0, 0, 16, 224, 112, 120,
      128, 136, 96, 120, 0, 0, 0, 0, 56, 88, 32, 104, 16, 208, 104, 248,
      24, 128, 160, 160, 88, 136, 40, 104, 112, 240, 96, 256, 32, 136, 40, 56,
      8, 128, 48, 160, 24, 216, 136, 160, 160, 160, 48, 112, 0, 0, 0, 0,
      0, 0, 0, 0, 200, 224, 72, 248, 16, 40, 0, 192, 120, 176, 40, 160,
      0, 0, 0, 0, 224, 248, 32, 64, 176, 240, 144, 248, 72, 128, 56, 200,
      128, 176, 56, 192, 248, 256, 0, 160, 24, 176, 112, 112, 24, 32, 0, 112,
      64, 232, 24, 144, 24, 56, 16, 64, 240, 256, 8, 128, 200, 200, 72, 240,
      80, 136, 160, 208, 72, 192, 32, 96, 8, 208, 128, 128, 176, 256, 24, 112,
      96, 224, 136, 136, 48, 144, 56, 104, 8, 136, 56, 160, 160, 248, 24, 56,
      0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 80, 168, 112, 240,
      72, 192, 144, 224, 224, 256, 32, 120, 208, 216, 96, 200, 120, 240, 48, 56,
      56, 176, 112, 136, 96, 240, 208, 208, 216, 256, 48, 168, 40, 200, 72, 112,
      96, 112, 144, 168, 40, 80, 48, 176, 40, 104, 80, 176, 16, 16, 88, 256,
      56, 224, 64, 248, 176, 248, 192, 224, 8, 176, 16, 168, 0, 0, 0, 0,
      0, 0, 0, 0, 96, 112, 176, 208, 72, 120, 152, 224, 40, 96, 176, 216,
      32, 240, 24, 200, 0, 0, 0, 0, 80, 168, 120, 144, 24, 120, 8, 32,
      8, 168, 32, 128, 128, 192, 80, 176, 16, 200, 208, 256, 112, 240, 104, 224,
      176, 184, 32, 216, 176, 200, 112, 216, 152, 176, 112, 200, 0, 0, 0, 0,
      80, 168, 24, 208, 8, 72, 120, 200, 24, 208, 72, 88, 136, 160, 152, 176,
      0, 0, 0, 0, 32, 208, 152, 176, 112, 240, 16, 216, 160, 168, 24, 136,
      16, 160, 88, 120, 0, 0, 0, 0, 88, 104, 80, 232, 72, 200, 184, 216,
      144, 152, 48, 96, 72, 232, 104, 168, 0, 0, 0, 0, 72, 232, 144, 160,
      128, 168, 112, 200, 40, 128, 160, 168, 0, 0, 0, 0, 0, 0, 0, 0,
      32, 32, 0, 40, 80, 224, 24, 200, 160, 208, 64, 104, 80, 224, 112, 152,
      24, 208, 96, 256, 32, 240, 8, 136, 128, 192, 24, 144, 112, 168, 192, 224,
      16, 80, 48, 88, 0, 0, 0, 0, 184, 248, 152, 224, 64, 120, 32, 184,
      32, 56, 160, 224, 128, 240, 80, 200, 128, 256, 0, 80, 104, 224, 152, 192,
      136, 192, 40, 144, 32, 208, 40, 240, 24, 72, 40, 152, 0, 0, 0, 0,
      8, 208, 56, 80, 128, 208, 48, 96, 184, 240, 152, 200, 120, 160, 8, 248,
      64, 256, 0, 56, 112, 152, 16, 72, 112, 200, 184, 192, 160, 216, 168, 240,
      24, 248, 16, 224, 0, 0, 0, 0, 120, 168, 24, 64, 88, 200, 16, 208,
      32, 128, 160, 248, 88, 112, 16, 192, 96, 256, 152, 192, 88, 248, 8, 192,
      120, 160, 32, 48, 192, 248, 160, 176, 24, 208, 104, 224, 0, 0, 0, 0};
  alignas(16) static constexpr uint16_t kTm[896] = {
      2608, 1504, 1520, 464, 1368, 848, 608, 2352, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2960, 2736, 3176, 472,
      2584, 2976, 552, 672, 2632, 1264, 1376, 520, 2544, 2928, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1280, 912, 3464, 3464, 560, 2624, 2872, 1120,
      3488, 1272, 3288, 2600, 2896, 3256, 504, 768, 696, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 432, 3336, 952, 1384, 2400, 3168, 2888, 3536, 1136, 512, 2992, 3320,
      1176, 728, 2880, 864, 2720, 2656, 3304, 720, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      736, 680, 2376, 2520, 3072, 312, 776, 344, 320, 3040, 928, 3224, 2512, 2512, 1400, 872,
      672, 2656, 3376, 2488, 3048, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1048, 1088, 328, 3208,
      2360, 2968, 1104, 464, 3016, 2440, 2896, 2952, 744, 304, 1000, 1256, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 640, 2344, 1408, 2672, 752, 960, 536, 776,
      2320, 1240, 1096, 904, 584, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 640, 856, 3088, 328, 624, 3168, 1136, 2368, 3040, 2944, 1520, 496,
      880, 2448, 1112, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2784, 3096, 976, 1120, 1056, 512, 344, 2328, 3568, 288, 792, 2912, 400, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2752, 1048, 2904, 3192,
      2504, 560, 2736, 2712, 360, 3264, 944, 2336, 392, 2920, 2600, 504, 592, 3304, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2480, 1040, 3280, 2464, 1160, 1184, 3120, 2936,
      1504, 3288, 2952, 1248, 448, 496, 2664, 2768, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 3328, 3136, 1416, 2368, 944, 1240, 1208, 2816, 2496, 2568, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2416, 544, 752, 384, 960, 2968, 1488, 3200, 2696, 1344, 1080, 872, 3584, 808, 2456, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1288, 1088, 976, 624,
      576, 3208, 2536, 320, 1216, 424, 2496, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 296, 3328, 712, 1232, 1384, 544, 2808, 352,
      352, 824, 888, 1192, 2360, 3104, 2848, 896, 2472, 2696, 3392, 392, 1096, 2552, 3032, 608,
      2744, 2456, 936, 1552, 2784, 2688, 688, 2712, 416, 824, 3152, 2824, 2560, 800, 1080, 1400,
      1208, 2720, 3312, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2904, 2760, 2832, 2800, 1128, 1128, 3232, 1072, 3072, 928, 3552, 288, 3016, 3128, 2776, 2880,
      3296, 2632, 3376, 1376, 3160, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 368, 368, 3136, 784,
      952, 2376, 472, 536, 840, 800, 280, 896, 2320, 3128, 2840, 552, 2792, 1328, 2928, 3248,
      2664, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1144, 456, 416, 2672, 3008, 600, 648, 728,
      864, 744, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 296, 1232, 664, 480, 488, 3008, 3240, 1008, 2552, 1536, 304, 440,
      1200, 1256, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      3088, 784, 1032, 3000, 456, 3024, 1072, 1024, 1056, 3064, 840, 1104, 3184, 2824, 992, 2336,
      968, 1368, 3144, 3144, 832, 832, 3256, 584, 3312, 880, 3248, 616, 2344, 2480, 816, 3096,
      912, 2760, 1408, 2832, 3000, 2464, 2936, 1016, 2560, 1216, 2976, 968, 648, 3032, 2856, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2728, 2960, 1032, 3432, 2400, 1160, 1184, 3240,
      312, 2648, 920, 3152, 2944, 904, 440, 408, 2984, 1200, 3160, 2704, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 736, 2728, 704, 2528, 760, 3104, 3056, 2848, 2840, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1280, 3192, 3080, 2592, 760, 488, 3232, 2776, 2920, 848, 984, 2792, 520, 1536, 1112, 656,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2752, 816, 856, 712,
      688, 2808, 384, 1192, 1008, 2408, 2408, 3488, 280, 1176, 2440, 792, 2816, 1248, 2984, 2640,
      720, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 432, 3336, 2864, 2608, 3024, 2624, 2800, 3176,
      2432, 3536, 1440, 2992, 2328, 1152, 1152, 768, 2544, 2488, 408, 3048, 616, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 680, 704, 3456, 2592, 2432, 2584, 3064, 2888, 920, 696, 2856, 2352,
      936, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2416, 1288, 2864, 1144, 1040, 3280, 664, 480, 2872, 2536, 2392, 992, 1272, 424, 3448, 984,
      808, 2640, 2448, 2768, 656, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2504, 3264, 2912, 448,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2688, 2520, 888, 1016, 2648, 3056, 360, 3224,
      3200, 2472, 272, 3392, 2744, 3296, 3424, 1000, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 3080, 2528, 576, 3120, 1024, 600, 3184, 2392, 3320, 272, 3416, 1264,
      2568, 592, 400, 2704, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552};
  struct Lane {
    double kf[R], kr[R];
    double W[S], iW[S];
    double rho, irho;
    uint32_t op[R][4], tm[kTermLen];   // LDS addresses, formed once per system
    uint32_t c_at;
  };
  __device__ __attribute__((noinline)) static void rates(Params p, double T, double* lds, int r) {
    const double lnT = crm::cr_log(T);
    double* const Q = lds + kOffQ;
#pragma nounroll
    for (int m = 0; m < R; ++m) {
      const int j = kRxOf[m * kL + r];
      Q[m * kL + r] = j >= 0 ? crm::cr_exp(p[j] + p[NR + j] * lnT - p[2 * NR + j] / T) : 0.0;
    }
  }
  __device__ static void init(Lane& L, const Params& p, const double* __restrict__ g, int64_t i,
                              int64_t n, const Grp<WNet>& x) {
    double* const Q = x.lds + kOffQ;
    rates(p, g[i], x.lds, x.r);
#pragma unroll
    for (int m = 0; m < R; ++m) {
      const int j = kRxOf[m * kL + x.r];
      L.kf[m] = Q[m * kL + x.r];
      L.kr[m] = j >= 0 ? L.kf[m] * p[3 * NR + j] : 0.0;
    }
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
  }
};

}  // namespace gen_n32r133_bcb31e07

template <>
struct FastVariant<gen_n32r133_bcb31e07::Net> {
  using type = gen_n32r133_bcb31e07::GNet;
};

}  // namespace rkmi
