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
  // three waves per SIMD: the evaluation loop fits 168 registers (the power
  // method and the set-up of a system run out of line)
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
  static constexpr int kTermBits = 9;
  static constexpr int kTermsPerWord = 3;
  static constexpr int kTermWords = 14;
  static constexpr int kTermLen = 40;
  static constexpr int kChunk = 4;
  using Params = const double*;
  static constexpr int kSp[32] = {
      20, 0, 4, 18, 11, 13, 26, 28, 3, 22, 21, 15, 12, 5, 10, 24,
      29, 14, 23, 16, 17, 25, 27, 8, 6, 19, 1, 9, 2, 7, 31, 30};
  static constexpr int16_t kRxOf[144] = {
      0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15,
      16, 19, 20, 21, 22, 23, 24, 26, 27, 28, 29, 30, 31, 32, 33, 34,
      35, 36, 37, 38, 39, 40, 41, 42, 43, 44, 45, 46, 47, 48, 49, 50,
      51, 52, 53, 54, 55, 56, 57, 59, 60, 61, 62, 63, 64, 65, 67, 68,
      69, 70, 71, 72, 73, 74, 75, 76, 78, 80, 81, 82, 83, 84, 85, 87,
      89, 91, 92, 93, 94, 95, 96, 97, 98, 99, 100, 101, 102, 103, 104, 105,
      106, 107, 108, 109, 110, 111, 112, 115, 117, 118, 119, 120, 121, 122, 123, 124,
      125, 126, 127, 128, 129, 130, 131, 132, -1, -1, -1, -1, -1, -1, -1, -1,
      17, 18, 25, 58, 66, 77, 79, 86, 88, 90, 113, 114, 116, -1, -1, -1};
  // lane r's operand codes and packed term codes, each lane's contiguous and
  // 16-byte aligned (read as whole vectors at every evaluation)
  static constexpr int kRxWords = 12;
  static constexpr int kTcWords = 16;
  alignas(16) static constexpr uint32_t kRx[192] = {
      386141960, 470422535, 520952322, 285612801, 471074564, 184945154, 234882051, 370349073, 537592322, 0, 0, 0, 117841423, 336663824, 235804163, 369364485,
      185145859, 235477253, 453123598, 437522698, 352722971, 0, 0, 0, 286333964, 370417432, 201726480, 336074510, 286201614, 235279380, 302323729, 520690713,
      235085846, 0, 0, 0, 453252886, 285414676, 269490689, 504699668, 469901059, 302192656, 420093456, 520625159, 537664003, 0, 0, 0,
      454498569, 336731401, 369757445, 521281046, 420551176, 419960593, 487197963, 319097091, 538581250, 0, 0, 0, 319689990, 319691786, 252582914, 336665347,
      268702977, 201594889, 335941633, 403117584, 167780368, 0, 0, 0, 436409610, 117772548, 403905549, 454429701, 419634692, 285280514, 520164367, 419634186,
      117448712, 0, 0, 0, 470620675, 235674392, 420223770, 335877647, 286135815, 336859139, 402726667, 471342870, 537665038, 0, 0, 0,
      420813850, 151132672, 369760272, 117645076, 437919244, 402654466, 470555413, 0, 251928604, 0, 0, 0, 151328008, 420415745, 336600842, 100930575,
      470621710, 252384258, 168237569, 0, 335552543, 0, 0, 0, 402787851, 471011081, 285285892, 420683287, 83887108, 151130894, 336007425, 0,
      537989124, 0, 0, 0, 419893257, 218634772, 201724690, 503912729, 268964873, 302193928, 319101696, 0, 268509214, 0, 0, 0,
      470947849, 471015191, 134350595, 134419727, 522064134, 369494533, 370350596, 0, 403906572, 0, 0, 0, 218435851, 302978314, 504239370, 134487836,
      353636357, 67178243, 437653004, 0, 0, 0, 0, 0, 352458241, 404166926, 521408516, 218368775, 353504780, 436345099, 453908758, 0,
      0, 0, 0, 0, 420353296, 218567174, 420353555, 353180937, 252449040, 471340302, 503650820, 0, 0, 0, 0, 0};
  alignas(16) static constexpr uint32_t kTc[256] = {
      4727490, 53749957, 13130793, 14445285, 16897770, 35953405, 22939908, 26613335, 76076312, 63278193, 37800205, 37822608, 37822608, 144, 0, 0,
      35195594, 23138890, 1456736, 5512892, 54537858, 9716257, 59530797, 18737380, 82182395, 70296657, 72139025, 37805343, 37822608, 144, 0, 0,
      52430336, 12959964, 16284217, 65047282, 35780860, 71875157, 75906364, 37822608, 1141248, 59784398, 68806892, 37822608, 37822608, 144, 0, 0,
      7612428, 13744849, 23897678, 37822562, 51217085, 9193172, 58741466, 19820101, 68551423, 73280265, 77403964, 37822608, 37822608, 144, 0, 0,
      33652412, 21005040, 73015385, 37822745, 50070530, 52438545, 13918250, 18647106, 68813566, 36317270, 76432668, 37822608, 37822608, 144, 0, 0,
      7084551, 56115231, 16547032, 37891145, 2887862, 54538767, 15228455, 81386221, 67931204, 26091604, 31082784, 37822608, 37822608, 144, 0, 0,
      48853510, 55155402, 56994516, 63768885, 18911478, 75118174, 29770349, 37822608, 80480259, 59355849, 14274277, 74855521, 37822574, 144, 0, 0,
      48762548, 52174860, 56375322, 16899800, 82350659, 76599391, 31346981, 37822608, 7173810, 15754284, 81914941, 70559819, 37822579, 144, 0, 0,
      5075462, 58304130, 14838503, 64349756, 69510726, 71966299, 322854, 54854327, 12604962, 21101625, 26523730, 37822608, 37822608, 144, 0, 0,
      4817077, 9545524, 12960296, 61107430, 28358905, 29507693, 1463079, 7353365, 59095590, 36837434, 29415531, 37822580, 37822608, 144, 0, 0,
      2191543, 50601147, 51742337, 13483727, 64782062, 71605325, 50405658, 11119307, 22671074, 26881629, 74239627, 37822748, 37822608, 144, 0, 0,
      6645426, 9714380, 62510825, 35692098, 73539161, 2452624, 52001981, 53581336, 17162811, 68985597, 29930760, 37822758, 37822608, 144, 0, 0,
      8924852, 60839463, 67236995, 22322823, 75288894, 3675280, 6448434, 11644626, 67667766, 70128904, 25476186, 37822608, 37822608, 144, 0, 0,
      5773833, 60933846, 66884663, 70915331, 29152866, 2884212, 8137922, 62943454, 35255026, 76862569, 37822581, 37822608, 37822608, 144, 0, 0,
      52175032, 10504399, 34979547, 26090754, 76337764, 54102312, 12170784, 62772276, 82614517, 30028390, 37900915, 37822608, 37822608, 144, 0, 0,
      51477514, 9977033, 69077722, 72400472, 30742631, 57763447, 60319277, 65042156, 20051706, 72755001, 37805885, 37822608, 37822608, 144, 0, 0};
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
  static constexpr int kMaxRkck = 64;
  static constexpr int kMaxRkc = 24;
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
      0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15,
      16, 19, 20, 21, 22, 23, 24, 26, 27, 28, 29, 30, 31, 32, 33, 34,
      35, 36, 37, 38, 39, 40, 41, 42, 43, 44, 45, 46, 47, 48, 49, 50,
      51, 52, 53, 54, 55, 56, 57, 59, 60, 61, 62, 63, 64, 65, 67, 68,
      69, 70, 71, 72, 73, 74, 75, 76, 78, 80, 81, 82, 83, 84, 85, 87,
      89, 91, 92, 93, 94, 95, 96, 97, 98, 99, 100, 101, 102, 103, 104, 105,
      106, 107, 108, 109, 110, 111, 112, 115, 117, 118, 119, 120, 121, 122, 123, 124,
      125, 126, 127, 128, 129, 130, 131, 132, -1, -1, -1, -1, -1, -1, -1, -1,
      17, 18, 25, 58, 66, 77, 79, 86, 88, 90, 113, 114, 116, -1, -1, -1,
      -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1};
  // LDS byte offsets within the system's area: each lane's rate operands
  // (R x 4), and the signed rates of its species in reaction order
  alignas(16) static constexpr uint16_t kOp[640] = {
      64, 120, 32, 184, 16, 208, 104, 248, 32, 56, 160, 224, 24, 32, 0, 112,
      16, 16, 88, 256, 120, 240, 48, 56, 24, 176, 112, 112, 24, 208, 72, 88,
      112, 240, 16, 216, 216, 256, 48, 168, 96, 224, 136, 136, 128, 208, 48, 96,
      112, 184, 120, 136, 136, 192, 40, 144, 176, 256, 24, 112, 176, 184, 32, 216,
      8, 208, 128, 128, 24, 248, 16, 224, 128, 240, 80, 200, 24, 208, 96, 256,
      72, 200, 184, 216, 40, 104, 80, 176, 64, 208, 136, 200, 88, 104, 80, 232,
      16, 200, 208, 256, 48, 168, 112, 152, 16, 224, 112, 120, 8, 168, 32, 128,
      8, 128, 48, 160, 128, 256, 0, 80, 80, 168, 24, 208, 104, 224, 152, 192,
      32, 240, 24, 200, 120, 160, 8, 248, 64, 256, 0, 56, 24, 208, 104, 224,
      208, 216, 96, 200, 56, 176, 112, 136, 88, 248, 8, 192, 112, 240, 96, 256,
      208, 224, 168, 200, 128, 192, 80, 176, 96, 240, 208, 208, 168, 216, 96, 224,
      224, 256, 32, 120, 64, 168, 40, 72, 80, 248, 128, 160, 112, 240, 104, 224,
      8, 208, 56, 80, 248, 256, 0, 160, 88, 112, 16, 192, 32, 240, 8, 136,
      32, 32, 0, 40, 8, 136, 56, 160, 32, 128, 136, 256, 72, 128, 56, 200,
      144, 152, 48, 96, 72, 160, 64, 128, 0, 216, 40, 152, 240, 256, 8, 128,
      72, 192, 144, 224, 24, 56, 16, 64, 48, 136, 240, 248, 32, 208, 152, 176,
      96, 256, 152, 192, 88, 136, 40, 104, 80, 168, 112, 240, 40, 128, 160, 168,
      96, 112, 176, 208, 0, 0, 0, 0, 8, 176, 16, 168, 32, 128, 160, 248,
      96, 112, 144, 168, 176, 200, 112, 216, 0, 0, 0, 0, 128, 168, 112, 200,
      152, 176, 112, 200, 128, 136, 96, 120, 32, 208, 40, 240, 0, 0, 0, 0,
      56, 160, 80, 224, 8, 216, 48, 136, 16, 80, 48, 88, 136, 160, 152, 176,
      0, 0, 0, 0, 128, 168, 136, 160, 40, 112, 32, 176, 40, 200, 72, 112,
      80, 136, 160, 208, 0, 0, 0, 0, 192, 248, 160, 176, 112, 184, 64, 160,
      160, 160, 48, 112, 200, 224, 72, 248, 0, 0, 0, 0, 160, 168, 24, 136,
      160, 216, 168, 240, 128, 192, 24, 144, 56, 224, 64, 248, 0, 0, 0, 0,
      72, 232, 144, 160, 176, 240, 144, 248, 136, 184, 64, 200, 24, 72, 40, 152,
      0, 0, 0, 0, 80, 224, 112, 152, 24, 216, 136, 160, 72, 192, 32, 96,
      128, 176, 56, 192, 0, 0, 0, 0, 32, 136, 40, 56, 40, 96, 176, 216,
      16, 72, 8, 136, 80, 224, 24, 200, 0, 0, 0, 0, 192, 216, 96, 112,
      120, 176, 40, 160, 24, 128, 160, 160, 176, 248, 192, 224, 0, 0, 0, 0,
      0, 208, 16, 72, 160, 248, 24, 56, 16, 40, 0, 192, 0, 0, 0, 0,
      0, 0, 0, 0, 8, 72, 120, 200, 120, 160, 32, 48, 16, 160, 88, 120,
      0, 0, 0, 0, 0, 0, 0, 0, 72, 120, 152, 224, 184, 240, 152, 200,
      112, 152, 16, 72, 0, 0, 0, 0, 0, 0, 0, 0, 160, 208, 64, 104,
      200, 200, 72, 240, 64, 232, 24, 144, 0, 0, 0, 0, 0, 0, 0, 0,
      184, 248, 152, 224, 120, 168, 24, 64, 40, 80, 48, 176, 0, 0, 0, 0,
      0, 0, 0, 0, 80, 168, 120, 144, 224, 248, 32, 64, 24, 120, 8, 32,
      0, 0, 0, 0, 0, 0, 0, 0, 112, 200, 184, 192, 56, 88, 32, 104,
      88, 200, 16, 208, 0, 0, 0, 0, 0, 0, 0, 0, 48, 144, 56, 104,
      72, 232, 104, 168, 112, 168, 192, 224, 0, 0, 0, 0, 0, 0, 0, 0};
  alignas(16) static constexpr uint16_t kTm[896] = {
      2512, 1336, 1344, 864, 1368, 976, 1040, 3176, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2432, 2520, 2600, 608,
      2704, 2872, 960, 1016, 3128, 1088, 1384, 1096, 3160, 3168, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 352, 384, 3344, 3344, 464, 2576, 2616, 624,
      3376, 808, 2960, 3008, 3024, 3032, 992, 1024, 1048, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 320, 2376, 424, 1312, 2584, 2672, 2744, 3368, 720, 752, 2840, 2856,
      832, 936, 3016, 1000, 3064, 3088, 3248, 1216, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      272, 296, 2496, 2656, 2688, 664, 728, 760, 768, 2832, 824, 2880, 2912, 2912, 1360, 952,
      1016, 3088, 3424, 3184, 3208, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 344, 376, 448, 2608,
      2712, 2752, 712, 864, 2936, 2968, 3024, 3056, 1056, 1128, 1160, 1200, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 280, 2360, 1304, 2568, 544, 616, 656, 728,
      2928, 912, 928, 1008, 1080, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 280, 360, 2448, 448, 520, 2672, 720, 2816, 2832, 2888, 1344, 1112,
      1120, 3240, 1208, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2320, 2392, 488, 624, 672, 752, 760, 2864, 3392, 872, 944, 3048, 1192, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2352, 344, 2408, 2416,
      2480, 464, 2520, 2528, 744, 2824, 792, 2920, 920, 3000, 3008, 992, 1184, 3248, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2368, 400, 2488, 2552, 560, 592, 2648, 2680,
      1336, 2960, 3056, 1064, 1072, 1112, 3224, 3264, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 2400, 2424, 1296, 2816, 792, 912, 984, 3072, 3120, 3144, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2336, 456, 544, 584, 616, 2752, 1320, 2896, 2944, 1352, 904, 952, 3440, 1104, 3192, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 328, 376, 488, 520,
      528, 2608, 2624, 768, 776, 856, 3120, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 312, 2400, 392, 440, 1312, 456, 2560, 536,
      536, 568, 632, 648, 2712, 2720, 2848, 840, 2904, 2944, 3400, 920, 928, 3040, 3080, 1040,
      3096, 3192, 1152, 1552, 2320, 2328, 472, 2528, 504, 568, 2760, 2776, 2800, 800, 904, 1360,
      984, 3064, 3136, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2408, 2440, 2456, 2592, 552, 552, 2640, 600, 2688, 824, 3384, 872, 2936, 2952, 2984, 3016,
      3112, 3128, 3424, 1384, 3256, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 288, 288, 2424, 408,
      424, 2496, 608, 656, 696, 800, 816, 840, 2928, 2952, 2992, 960, 3104, 1376, 3168, 3216,
      3224, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 368, 432, 504, 2568, 2664, 688, 896, 936,
      1000, 1056, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 312, 440, 480, 496, 576, 2664, 2696, 736, 3040, 1392, 1128, 1136,
      1168, 1200, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2448, 408, 416, 2472, 432, 2536, 600, 640, 672, 2728, 696, 712, 2768, 2776, 784, 2920,
      888, 1368, 2976, 2976, 968, 968, 3032, 1080, 3136, 1120, 3216, 1176, 2360, 2368, 336, 2392,
      384, 2440, 1304, 2456, 2472, 2552, 2680, 680, 2800, 776, 2872, 888, 896, 3080, 3152, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2344, 2432, 416, 3360, 2584, 560, 592, 2696,
      664, 2736, 704, 2760, 2888, 1008, 1136, 1144, 3200, 1168, 3256, 3272, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 272, 2344, 304, 2544, 512, 2720, 2784, 2848, 2992, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      352, 2416, 2464, 2504, 512, 576, 2640, 2984, 3000, 976, 1032, 3104, 1096, 1392, 1208, 1224,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2352, 336, 360, 392,
      472, 2560, 584, 648, 736, 2792, 2792, 3376, 816, 832, 2968, 944, 3072, 1064, 3200, 3232,
      1216, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 320, 2376, 2384, 2512, 2536, 2576, 2592, 2600,
      2632, 3368, 1328, 2840, 2864, 848, 848, 1024, 3160, 3184, 1144, 3208, 1176, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 296, 304, 3352, 2504, 2632, 2704, 2728, 2744, 704, 1048, 3152, 3176,
      1152, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      2336, 328, 2384, 368, 400, 2488, 480, 496, 2616, 2624, 2808, 784, 808, 856, 3408, 1032,
      1104, 3232, 3240, 3264, 1224, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2480, 2824, 3048, 1072,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 2328, 2656, 632, 680, 2736, 2784, 744, 2880,
      2896, 2904, 880, 3400, 3096, 3112, 3432, 1160, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552,
      1552, 1552, 1552, 1552, 2464, 2544, 528, 2648, 640, 688, 2768, 2808, 2856, 880, 3416, 1088,
      3144, 1184, 1192, 3272, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552, 1552};
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
