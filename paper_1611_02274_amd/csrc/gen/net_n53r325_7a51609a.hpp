// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Mass-action network: 53 species, 325 reversible reactions (topology n53r325_7a51609a).
#pragma once

#include "../rk_adjoint.hpp"
#include "../rk_group.hpp"

namespace rkmi {
namespace gen_n53r325_7a51609a {

struct Net {
  static constexpr int N = 53;
  static constexpr int NR = 325;
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
    q = (kf * C[16]) * C[48] - (kr * C[7]) * C[31];
    om[16] -= q;
    om[48] -= q;
    om[7] += q;
    om[31] += q;
    kf = L.kf[1 * kLdsStride];
    kr = kf * ld_uniform(iK, 1);
    q = (kf * C[13]) * C[26] - (kr * C[16]) * C[31];
    om[13] -= q;
    om[26] -= q;
    om[16] += q;
    om[31] += q;
    kf = L.kf[2 * kLdsStride];
    kr = kf * ld_uniform(iK, 2);
    q = (kf * C[9]) * C[45] - (kr * C[19]) * C[33];
    om[9] -= q;
    om[45] -= q;
    om[19] += q;
    om[33] += q;
    kf = L.kf[3 * kLdsStride];
    kr = kf * ld_uniform(iK, 3);
    q = (kf * C[17]) * C[34] - (kr * C[5]) * C[51];
    om[17] -= q;
    om[34] -= q;
    om[5] += q;
    om[51] += q;
    kf = L.kf[4 * kLdsStride];
    kr = kf * ld_uniform(iK, 4);
    q = (kf * C[5]) * C[37] - (kr * C[19]) * C[28];
    om[5] -= q;
    om[37] -= q;
    om[19] += q;
    om[28] += q;
    kf = L.kf[5 * kLdsStride];
    kr = kf * ld_uniform(iK, 5);
    q = (kf * C[1]) * C[38] - (kr * C[7]) * C[25];
    om[1] -= q;
    om[38] -= q;
    om[7] += q;
    om[25] += q;
    kf = L.kf[6 * kLdsStride];
    kr = kf * ld_uniform(iK, 6);
    q = (kf * C[9]) * C[32] - (kr * C[22]) * C[44];
    om[9] -= q;
    om[32] -= q;
    om[22] += q;
    om[44] += q;
    kf = L.kf[7 * kLdsStride];
    kr = kf * ld_uniform(iK, 7);
    q = (kf * C[14]) * C[40] - (kr * C[11]) * C[27];
    om[14] -= q;
    om[40] -= q;
    om[11] += q;
    om[27] += q;
    kf = L.kf[8 * kLdsStride];
    kr = kf * ld_uniform(iK, 8);
    q = (kf * C[18]) * M - (kr * C[7]) * C[14];
    om[18] -= q;
    om[7] += q;
    om[14] += q;
    kf = L.kf[9 * kLdsStride];
    kr = kf * ld_uniform(iK, 9);
    q = (kf * C[16]) * C[24] - (kr * C[11]) * C[31];
    om[16] -= q;
    om[24] -= q;
    om[11] += q;
    om[31] += q;
    kf = L.kf[10 * kLdsStride];
    kr = kf * ld_uniform(iK, 10);
    q = (kf * C[24]) * C[31] - (kr * C[39]) * C[43];
    om[24] -= q;
    om[31] -= q;
    om[39] += q;
    om[43] += q;
    kf = L.kf[11 * kLdsStride];
    kr = kf * ld_uniform(iK, 11);
    q = (kf * C[8]) * C[35] - (kr * C[16]) * C[16];
    om[8] -= q;
    om[35] -= q;
    om[16] += q;
    om[16] += q;
    kf = L.kf[12 * kLdsStride];
    kr = kf * ld_uniform(iK, 12);
    q = (kf * C[10]) * C[39] - (kr * C[32]) * C[50];
    om[10] -= q;
    om[39] -= q;
    om[32] += q;
    om[50] += q;
    kf = L.kf[13 * kLdsStride];
    kr = kf * ld_uniform(iK, 13);
    q = (kf * C[33]) * C[52] - (kr * C[31]) * C[47];
    om[33] -= q;
    om[52] -= q;
    om[31] += q;
    om[47] += q;
    kf = L.kf[14 * kLdsStride];
    kr = kf * ld_uniform(iK, 14);
    q = (kf * C[13]) * C[13] - (kr * C[7]) * C[35];
    om[13] -= q;
    om[13] -= q;
    om[7] += q;
    om[35] += q;
    kf = L.kf[15 * kLdsStride];
    kr = kf * ld_uniform(iK, 15);
    q = (kf * C[28]) * C[46] - (kr * C[8]) * C[37];
    om[28] -= q;
    om[46] -= q;
    om[8] += q;
    om[37] += q;
    kf = L.kf[16 * kLdsStride];
    kr = kf * ld_uniform(iK, 16);
    q = (kf * C[7]) * C[42] - (kr * C[9]) * C[28];
    om[7] -= q;
    om[42] -= q;
    om[9] += q;
    om[28] += q;
    kf = L.kf[17 * kLdsStride];
    kr = kf * ld_uniform(iK, 17);
    q = (kf * C[14]) * C[14] - (kr * C[19]) * C[40];
    om[14] -= q;
    om[14] -= q;
    om[19] += q;
    om[40] += q;
    kf = L.kf[18 * kLdsStride];
    kr = kf * ld_uniform(iK, 18);
    q = (kf * C[14]) * C[17] - (kr * C[9]) * C[47];
    om[14] -= q;
    om[17] -= q;
    om[9] += q;
    om[47] += q;
    kf = L.kf[19 * kLdsStride];
    kr = kf * ld_uniform(iK, 19);
    q = (kf * C[8]) * C[30] - (kr * C[6]) * C[32];
    om[8] -= q;
    om[30] -= q;
    om[6] += q;
    om[32] += q;
    kf = L.kf[20 * kLdsStride];
    kr = kf * ld_uniform(iK, 20);
    q = (kf * C[37]) * C[52] - (kr * C[25]) * C[33];
    om[37] -= q;
    om[52] -= q;
    om[25] += q;
    om[33] += q;
    kf = L.kf[21 * kLdsStride];
    kr = kf * ld_uniform(iK, 21);
    q = (kf * C[11]) * C[12] - (kr * C[5]) * C[19];
    om[11] -= q;
    om[12] -= q;
    om[5] += q;
    om[19] += q;
    kf = L.kf[22 * kLdsStride];
    kr = kf * ld_uniform(iK, 22);
    q = (kf * C[4]) * C[47] - (kr * C[5]) * C[51];
    om[4] -= q;
    om[47] -= q;
    om[5] += q;
    om[51] += q;
    kf = L.kf[23 * kLdsStride];
    kr = kf * ld_uniform(iK, 23);
    q = (kf * C[14]) * C[36] - (kr * C[18]) * C[25];
    om[14] -= q;
    om[36] -= q;
    om[18] += q;
    om[25] += q;
    kf = L.kf[24 * kLdsStride];
    kr = kf * ld_uniform(iK, 24);
    q = (kf * C[24]) * C[33] - (kr * C[21]) * C[23];
    om[24] -= q;
    om[33] -= q;
    om[21] += q;
    om[23] += q;
    kf = L.kf[25 * kLdsStride];
    kr = kf * ld_uniform(iK, 25);
    q = (kf * C[2]) * C[25] - (kr * C[23]) * M;
    om[2] -= q;
    om[25] -= q;
    om[23] += q;
    kf = L.kf[26 * kLdsStride];
    kr = kf * ld_uniform(iK, 26);
    q = (kf * C[0]) * C[43] - (kr * C[13]) * C[16];
    om[0] -= q;
    om[43] -= q;
    om[13] += q;
    om[16] += q;
    kf = L.kf[27 * kLdsStride];
    kr = kf * ld_uniform(iK, 27);
    q = (kf * C[3]) * C[32] - (kr * C[12]) * C[43];
    om[3] -= q;
    om[32] -= q;
    om[12] += q;
    om[43] += q;
    kf = L.kf[28 * kLdsStride];
    kr = kf * ld_uniform(iK, 28);
    q = (kf * C[13]) * C[23] - (kr * C[34]) * C[44];
    om[13] -= q;
    om[23] -= q;
    om[34] += q;
    om[44] += q;
    kf = L.kf[29 * kLdsStride];
    kr = kf * ld_uniform(iK, 29);
    q = (kf * C[9]) * C[35] - (kr * C[37]) * C[40];
    om[9] -= q;
    om[35] -= q;
    om[37] += q;
    om[40] += q;
    kf = L.kf[30 * kLdsStride];
    kr = kf * ld_uniform(iK, 30);
    q = (kf * C[26]) * C[33] - (kr * C[23]) * C[32];
    om[26] -= q;
    om[33] -= q;
    om[23] += q;
    om[32] += q;
    kf = L.kf[31 * kLdsStride];
    kr = kf * ld_uniform(iK, 31);
    q = (kf * C[5]) * C[41] - (kr * C[30]) * C[42];
    om[5] -= q;
    om[41] -= q;
    om[30] += q;
    om[42] += q;
    kf = L.kf[32 * kLdsStride];
    kr = kf * ld_uniform(iK, 32);
    q = (kf * C[13]) * C[45] - (kr * C[37]) * C[52];
    om[13] -= q;
    om[45] -= q;
    om[37] += q;
    om[52] += q;
    kf = L.kf[33 * kLdsStride];
    kr = kf * ld_uniform(iK, 33);
    q = (kf * C[9]) * C[39] - (kr * C[10]) * C[52];
    om[9] -= q;
    om[39] -= q;
    om[10] += q;
    om[52] += q;
    kf = L.kf[34 * kLdsStride];
    kr = kf * ld_uniform(iK, 34);
    q = (kf * C[8]) * C[13] - (kr * C[0]) * C[15];
    om[8] -= q;
    om[13] -= q;
    om[0] += q;
    om[15] += q;
    kf = L.kf[35 * kLdsStride];
    kr = kf * ld_uniform(iK, 35);
    q = (kf * C[4]) * C[31] - (kr * C[12]) * C[43];
    om[4] -= q;
    om[31] -= q;
    om[12] += q;
    om[43] += q;
    kf = L.kf[36 * kLdsStride];
    kr = kf * ld_uniform(iK, 36);
    q = (kf * C[28]) * C[39] - (kr * C[42]) * C[45];
    om[28] -= q;
    om[39] -= q;
    om[42] += q;
    om[45] += q;
    kf = L.kf[37 * kLdsStride];
    kr = kf * ld_uniform(iK, 37);
    q = (kf * C[20]) * C[23] - (kr * C[36]) * C[50];
    om[20] -= q;
    om[23] -= q;
    om[36] += q;
    om[50] += q;
    kf = L.kf[38 * kLdsStride];
    kr = kf * ld_uniform(iK, 38);
    q = (kf * C[8]) * C[35] - (kr * C[5]) * C[36];
    om[8] -= q;
    om[35] -= q;
    om[5] += q;
    om[36] += q;
    kf = L.kf[39 * kLdsStride];
    kr = kf * ld_uniform(iK, 39);
    q = (kf * C[14]) * C[17] - (kr * C[12]) * C[13];
    om[14] -= q;
    om[17] -= q;
    om[12] += q;
    om[13] += q;
    kf = L.kf[40 * kLdsStride];
    kr = kf * ld_uniform(iK, 40);
    q = (kf * C[14]) * C[33] - (kr * C[31]) * C[50];
    om[14] -= q;
    om[33] -= q;
    om[31] += q;
    om[50] += q;
    kf = L.kf[41 * kLdsStride];
    kr = kf * ld_uniform(iK, 41);
    q = (kf * C[16]) * C[20] - (kr * C[10]) * C[13];
    om[16] -= q;
    om[20] -= q;
    om[10] += q;
    om[13] += q;
    kf = L.kf[42 * kLdsStride];
    kr = kf * ld_uniform(iK, 42);
    q = (kf * C[13]) * C[33] - (kr * C[16]) * C[48];
    om[13] -= q;
    om[33] -= q;
    om[16] += q;
    om[48] += q;
    kf = L.kf[43 * kLdsStride];
    kr = kf * ld_uniform(iK, 43);
    q = (kf * C[20]) * C[29] - (kr * C[18]) * C[19];
    om[20] -= q;
    om[29] -= q;
    om[18] += q;
    om[19] += q;
    kf = L.kf[44 * kLdsStride];
    kr = kf * ld_uniform(iK, 44);
    q = (kf * C[27]) * C[46] - (kr * C[16]) * C[51];
    om[27] -= q;
    om[46] -= q;
    om[16] += q;
    om[51] += q;
    kf = L.kf[45 * kLdsStride];
    kr = kf * ld_uniform(iK, 45);
    q = (kf * C[3]) * C[41] - (kr * C[8]) * C[30];
    om[3] -= q;
    om[41] -= q;
    om[8] += q;
    om[30] += q;
    kf = L.kf[46 * kLdsStride];
    kr = kf * ld_uniform(iK, 46);
    q = (kf * C[27]) * C[49] - (kr * C[31]) * C[47];
    om[27] -= q;
    om[49] -= q;
    om[31] += q;
    om[47] += q;
    kf = L.kf[47 * kLdsStride];
    kr = kf * ld_uniform(iK, 47);
    q = (kf * C[6]) * C[46] - (kr * C[2]) * C[16];
    om[6] -= q;
    om[46] -= q;
    om[2] += q;
    om[16] += q;
    kf = L.kf[48 * kLdsStride];
    kr = kf * ld_uniform(iK, 48);
    q = (kf * C[3]) * C[50] - (kr * C[0]) * C[6];
    om[3] -= q;
    om[50] -= q;
    om[0] += q;
    om[6] += q;
    kf = L.kf[49 * kLdsStride];
    kr = kf * ld_uniform(iK, 49);
    q = (kf * C[16]) * C[36] - (kr * C[18]) * C[33];
    om[16] -= q;
    om[36] -= q;
    om[18] += q;
    om[33] += q;
    kf = L.kf[50 * kLdsStride];
    kr = kf * ld_uniform(iK, 50);
    q = (kf * C[16]) * C[38] - (kr * C[8]) * C[36];
    om[16] -= q;
    om[38] -= q;
    om[8] += q;
    om[36] += q;
    kf = L.kf[51 * kLdsStride];
    kr = kf * ld_uniform(iK, 51);
    q = (kf * C[40]) * C[46] - (kr * C[9]) * C[23];
    om[40] -= q;
    om[46] -= q;
    om[9] += q;
    om[23] += q;
    kf = L.kf[52 * kLdsStride];
    kr = kf * ld_uniform(iK, 52);
    q = (kf * C[20]) * C[23] - (kr * C[0]) * C[21];
    om[20] -= q;
    om[23] -= q;
    om[0] += q;
    om[21] += q;
    kf = L.kf[53 * kLdsStride];
    kr = kf * ld_uniform(iK, 53);
    q = (kf * C[17]) * C[33] - (kr * C[12]) * C[44];
    om[17] -= q;
    om[33] -= q;
    om[12] += q;
    om[44] += q;
    kf = L.kf[54 * kLdsStride];
    kr = kf * ld_uniform(iK, 54);
    q = (kf * C[49]) * C[50] - (kr * C[27]) * C[37];
    om[49] -= q;
    om[50] -= q;
    om[27] += q;
    om[37] += q;
    kf = L.kf[55 * kLdsStride];
    kr = kf * ld_uniform(iK, 55);
    q = (kf * C[6]) * C[31] - (kr * C[14]) * C[29];
    om[6] -= q;
    om[31] -= q;
    om[14] += q;
    om[29] += q;
    kf = L.kf[56 * kLdsStride];
    kr = kf * ld_uniform(iK, 56);
    q = (kf * C[23]) * C[23] - (kr * C[34]) * C[49];
    om[23] -= q;
    om[23] -= q;
    om[34] += q;
    om[49] += q;
    kf = L.kf[57 * kLdsStride];
    kr = kf * ld_uniform(iK, 57);
    q = (kf * C[11]) * C[23] - (kr * C[14]) * C[22];
    om[11] -= q;
    om[23] -= q;
    om[14] += q;
    om[22] += q;
    kf = L.kf[58 * kLdsStride];
    kr = kf * ld_uniform(iK, 58);
    q = (kf * C[0]) * C[52] - (kr * C[1]) * C[23];
    om[0] -= q;
    om[52] -= q;
    om[1] += q;
    om[23] += q;
    kf = L.kf[59 * kLdsStride];
    kr = kf * ld_uniform(iK, 59);
    q = (kf * C[22]) * C[39] - (kr * C[15]) * C[52];
    om[22] -= q;
    om[39] -= q;
    om[15] += q;
    om[52] += q;
    kf = L.kf[60 * kLdsStride];
    kr = kf * ld_uniform(iK, 60);
    q = (kf * C[17]) * C[33] - (kr * C[7]) * C[45];
    om[17] -= q;
    om[33] -= q;
    om[7] += q;
    om[45] += q;
    kf = L.kf[61 * kLdsStride];
    kr = kf * ld_uniform(iK, 61);
    q = (kf * C[6]) * C[45] - (kr * C[40]) * C[47];
    om[6] -= q;
    om[45] -= q;
    om[40] += q;
    om[47] += q;
    kf = L.kf[62 * kLdsStride];
    kr = kf * ld_uniform(iK, 62);
    q = (kf * C[4]) * C[45] - (kr * C[9]) * C[52];
    om[4] -= q;
    om[45] -= q;
    om[9] += q;
    om[52] += q;
    kf = L.kf[63 * kLdsStride];
    kr = kf * ld_uniform(iK, 63);
    q = (kf * C[0]) * C[26] - (kr * C[4]) * C[49];
    om[0] -= q;
    om[26] -= q;
    om[4] += q;
    om[49] += q;
    kf = L.kf[64 * kLdsStride];
    kr = kf * ld_uniform(iK, 64);
    q = (kf * C[1]) * C[18] - (kr * C[20]) * C[27];
    om[1] -= q;
    om[18] -= q;
    om[20] += q;
    om[27] += q;
    kf = L.kf[65 * kLdsStride];
    kr = kf * ld_uniform(iK, 65);
    q = (kf * C[2]) * C[19] - (kr * C[12]) * C[50];
    om[2] -= q;
    om[19] -= q;
    om[12] += q;
    om[50] += q;
    kf = L.kf[66 * kLdsStride];
    kr = kf * ld_uniform(iK, 66);
    q = (kf * C[11]) * C[23] - (kr * C[18]) * C[34];
    om[11] -= q;
    om[23] -= q;
    om[18] += q;
    om[34] += q;
    kf = L.kf[67 * kLdsStride];
    kr = kf * ld_uniform(iK, 67);
    q = (kf * C[2]) * C[43] - (kr * C[14]) * C[16];
    om[2] -= q;
    om[43] -= q;
    om[14] += q;
    om[16] += q;
    kf = L.kf[68 * kLdsStride];
    kr = kf * ld_uniform(iK, 68);
    q = (kf * C[7]) * C[52] - (kr * C[16]) * C[51];
    om[7] -= q;
    om[52] -= q;
    om[16] += q;
    om[51] += q;
    kf = L.kf[69 * kLdsStride];
    kr = kf * ld_uniform(iK, 69);
    q = (kf * C[18]) * C[19] - (kr * C[21]) * C[50];
    om[18] -= q;
    om[19] -= q;
    om[21] += q;
    om[50] += q;
    kf = L.kf[70 * kLdsStride];
    kr = kf * ld_uniform(iK, 70);
    q = (kf * C[4]) * C[9] - (kr * C[3]) * C[10];
    om[4] -= q;
    om[9] -= q;
    om[3] += q;
    om[10] += q;
    kf = L.kf[71 * kLdsStride];
    kr = kf * ld_uniform(iK, 71);
    q = (kf * C[40]) * C[48] - (kr * C[9]) * C[39];
    om[40] -= q;
    om[48] -= q;
    om[9] += q;
    om[39] += q;
    kf = L.kf[72 * kLdsStride];
    kr = kf * ld_uniform(iK, 72);
    q = (kf * C[28]) * C[33] - (kr * C[8]) * C[36];
    om[28] -= q;
    om[33] -= q;
    om[8] += q;
    om[36] += q;
    kf = L.kf[73 * kLdsStride];
    kr = kf * ld_uniform(iK, 73);
    q = (kf * C[4]) * C[21] - (kr * C[15]) * C[19];
    om[4] -= q;
    om[21] -= q;
    om[15] += q;
    om[19] += q;
    kf = L.kf[74 * kLdsStride];
    kr = kf * ld_uniform(iK, 74);
    q = (kf * C[17]) * C[40] - (kr * C[3]) * C[33];
    om[17] -= q;
    om[40] -= q;
    om[3] += q;
    om[33] += q;
    kf = L.kf[75 * kLdsStride];
    kr = kf * ld_uniform(iK, 75);
    q = (kf * C[13]) * C[45] - (kr * C[19]) * C[49];
    om[13] -= q;
    om[45] -= q;
    om[19] += q;
    om[49] += q;
    kf = L.kf[76 * kLdsStride];
    kr = kf * ld_uniform(iK, 76);
    q = (kf * C[22]) * C[47] - (kr * C[3]) * C[31];
    om[22] -= q;
    om[47] -= q;
    om[3] += q;
    om[31] += q;
    kf = L.kf[77 * kLdsStride];
    kr = kf * ld_uniform(iK, 77);
    q = (kf * C[7]) * C[16] - (kr * C[14]) * C[20];
    om[7] -= q;
    om[16] -= q;
    om[14] += q;
    om[20] += q;
    kf = L.kf[78 * kLdsStride];
    kr = kf * ld_uniform(iK, 78);
    q = (kf * C[11]) * C[39] - (kr * C[15]) * C[27];
    om[11] -= q;
    om[39] -= q;
    om[15] += q;
    om[27] += q;
    kf = L.kf[79 * kLdsStride];
    kr = kf * ld_uniform(iK, 79);
    q = (kf * C[48]) * C[50] - (kr * C[7]) * C[25];
    om[48] -= q;
    om[50] -= q;
    om[7] += q;
    om[25] += q;
    kf = L.kf[80 * kLdsStride];
    kr = kf * ld_uniform(iK, 80);
    q = (kf * C[43]) * M - (kr * C[8]) * C[25];
    om[43] -= q;
    om[8] += q;
    om[25] += q;
    kf = L.kf[81 * kLdsStride];
    kr = kf * ld_uniform(iK, 81);
    q = (kf * C[10]) * C[50] - (kr * C[7]) * C[8];
    om[10] -= q;
    om[50] -= q;
    om[7] += q;
    om[8] += q;
    kf = L.kf[82 * kLdsStride];
    kr = kf * ld_uniform(iK, 82);
    q = (kf * C[17]) * C[34] - (kr * C[4]) * C[47];
    om[17] -= q;
    om[34] -= q;
    om[4] += q;
    om[47] += q;
    kf = L.kf[83 * kLdsStride];
    kr = kf * ld_uniform(iK, 83);
    q = (kf * C[9]) * C[12] - (kr * C[0]) * C[14];
    om[9] -= q;
    om[12] -= q;
    om[0] += q;
    om[14] += q;
    kf = L.kf[84 * kLdsStride];
    kr = kf * ld_uniform(iK, 84);
    q = (kf * C[2]) * C[35] - (kr * C[4]) * C[25];
    om[2] -= q;
    om[35] -= q;
    om[4] += q;
    om[25] += q;
    kf = L.kf[85 * kLdsStride];
    kr = kf * ld_uniform(iK, 85);
    q = (kf * C[24]) * C[46] - (kr * C[8]) * C[49];
    om[24] -= q;
    om[46] -= q;
    om[8] += q;
    om[49] += q;
    kf = L.kf[86 * kLdsStride];
    kr = kf * ld_uniform(iK, 86);
    q = (kf * C[25]) * C[35] - (kr * C[16]) * C[45];
    om[25] -= q;
    om[35] -= q;
    om[16] += q;
    om[45] += q;
    kf = L.kf[87 * kLdsStride];
    kr = kf * ld_uniform(iK, 87);
    q = (kf * C[9]) * C[26] - (kr * C[15]) * C[25];
    om[9] -= q;
    om[26] -= q;
    om[15] += q;
    om[25] += q;
    kf = L.kf[88 * kLdsStride];
    kr = kf * ld_uniform(iK, 88);
    q = (kf * C[7]) * C[18] - (kr * C[8]) * C[37];
    om[7] -= q;
    om[18] -= q;
    om[8] += q;
    om[37] += q;
    kf = L.kf[89 * kLdsStride];
    kr = kf * ld_uniform(iK, 89);
    q = (kf * C[33]) * C[50] - (kr * C[2]) * C[36];
    om[33] -= q;
    om[50] -= q;
    om[2] += q;
    om[36] += q;
    kf = L.kf[90 * kLdsStride];
    kr = kf * ld_uniform(iK, 90);
    q = (kf * C[2]) * C[43] - (kr * C[34]) * C[38];
    om[2] -= q;
    om[43] -= q;
    om[34] += q;
    om[38] += q;
    kf = L.kf[91 * kLdsStride];
    kr = kf * ld_uniform(iK, 91);
    q = (kf * C[22]) * C[51] - (kr * C[17]) * C[29];
    om[22] -= q;
    om[51] -= q;
    om[17] += q;
    om[29] += q;
    kf = L.kf[92 * kLdsStride];
    kr = kf * ld_uniform(iK, 92);
    q = (kf * C[43]) * M - (kr * C[3]) * C[36];
    om[43] -= q;
    om[3] += q;
    om[36] += q;
    kf = L.kf[93 * kLdsStride];
    kr = kf * ld_uniform(iK, 93);
    q = (kf * C[36]) * C[52] - (kr * C[33]) * C[39];
    om[36] -= q;
    om[52] -= q;
    om[33] += q;
    om[39] += q;
    kf = L.kf[94 * kLdsStride];
    kr = kf * ld_uniform(iK, 94);
    q = (kf * C[1]) * C[18] - (kr * C[9]) * C[25];
    om[1] -= q;
    om[18] -= q;
    om[9] += q;
    om[25] += q;
    kf = L.kf[95 * kLdsStride];
    kr = kf * ld_uniform(iK, 95);
    q = (kf * C[22]) * C[37] - (kr * C[10]) * C[35];
    om[22] -= q;
    om[37] -= q;
    om[10] += q;
    om[35] += q;
    kf = L.kf[96 * kLdsStride];
    kr = kf * ld_uniform(iK, 96);
    q = (kf * C[35]) * C[52] - (kr * C[27]) * C[31];
    om[35] -= q;
    om[52] -= q;
    om[27] += q;
    om[31] += q;
    kf = L.kf[97 * kLdsStride];
    kr = kf * ld_uniform(iK, 97);
    q = (kf * C[27]) * C[28] - (kr * C[24]) * C[50];
    om[27] -= q;
    om[28] -= q;
    om[24] += q;
    om[50] += q;
    kf = L.kf[98 * kLdsStride];
    kr = kf * ld_uniform(iK, 98);
    q = (kf * C[3]) * C[32] - (kr * C[18]) * C[27];
    om[3] -= q;
    om[32] -= q;
    om[18] += q;
    om[27] += q;
    kf = L.kf[99 * kLdsStride];
    kr = kf * ld_uniform(iK, 99);
    q = (kf * C[4]) * C[27] - (kr * C[12]) * C[40];
    om[4] -= q;
    om[27] -= q;
    om[12] += q;
    om[40] += q;
    kf = L.kf[100 * kLdsStride];
    kr = kf * ld_uniform(iK, 100);
    q = (kf * C[7]) * C[18] - (kr * C[28]) * C[46];
    om[7] -= q;
    om[18] -= q;
    om[28] += q;
    om[46] += q;
    kf = L.kf[101 * kLdsStride];
    kr = kf * ld_uniform(iK, 101);
    q = (kf * C[18]) * C[19] - (kr * C[5]) * C[44];
    om[18] -= q;
    om[19] -= q;
    om[5] += q;
    om[44] += q;
    kf = L.kf[102 * kLdsStride];
    kr = kf * ld_uniform(iK, 102);
    q = (kf * C[27]) * C[40] - (kr * C[23]) * C[34];
    om[27] -= q;
    om[40] -= q;
    om[23] += q;
    om[34] += q;
    kf = L.kf[103 * kLdsStride];
    kr = kf * ld_uniform(iK, 103);
    q = (kf * C[24]) * C[28] - (kr * C[11]) * C[21];
    om[24] -= q;
    om[28] -= q;
    om[11] += q;
    om[21] += q;
    kf = L.kf[104 * kLdsStride];
    kr = kf * ld_uniform(iK, 104);
    q = (kf * C[1]) * C[1] - (kr * C[51]) * M;
    om[1] -= q;
    om[1] -= q;
    om[51] += q;
    kf = L.kf[105 * kLdsStride];
    kr = kf * ld_uniform(iK, 105);
    q = (kf * C[4]) * C[49] - (kr * C[14]) * C[33];
    om[4] -= q;
    om[49] -= q;
    om[14] += q;
    om[33] += q;
    kf = L.kf[106 * kLdsStride];
    kr = kf * ld_uniform(iK, 106);
    q = (kf * C[23]) * C[41] - (kr * C[24]) * C[31];
    om[23] -= q;
    om[41] -= q;
    om[24] += q;
    om[31] += q;
    kf = L.kf[107 * kLdsStride];
    kr = kf * ld_uniform(iK, 107);
    q = (kf * C[16]) * C[32] - (kr * C[13]) * C[41];
    om[16] -= q;
    om[32] -= q;
    om[13] += q;
    om[41] += q;
    kf = L.kf[108 * kLdsStride];
    kr = kf * ld_uniform(iK, 108);
    q = (kf * C[1]) * C[20] - (kr * C[0]) * C[46];
    om[1] -= q;
    om[20] -= q;
    om[0] += q;
    om[46] += q;
    kf = L.kf[109 * kLdsStride];
    kr = kf * ld_uniform(iK, 109);
    q = (kf * C[6]) * C[45] - (kr * C[25]) * C[34];
    om[6] -= q;
    om[45] -= q;
    om[25] += q;
    om[34] += q;
    kf = L.kf[110 * kLdsStride];
    kr = kf * ld_uniform(iK, 110);
    q = (kf * C[9]) * C[48] - (kr * C[20]) * C[25];
    om[9] -= q;
    om[48] -= q;
    om[20] += q;
    om[25] += q;
    kf = L.kf[111 * kLdsStride];
    kr = kf * ld_uniform(iK, 111);
    q = (kf * C[13]) * C[48] - (kr * C[33]) * C[46];
    om[13] -= q;
    om[48] -= q;
    om[33] += q;
    om[46] += q;
    kf = L.kf[112 * kLdsStride];
    kr = kf * ld_uniform(iK, 112);
    q = (kf * C[12]) * C[38] - (kr * C[13]) * C[19];
    om[12] -= q;
    om[38] -= q;
    om[13] += q;
    om[19] += q;
    kf = L.kf[113 * kLdsStride];
    kr = kf * ld_uniform(iK, 113);
    q = (kf * C[1]) * C[9] - (kr * C[2]) * C[46];
    om[1] -= q;
    om[9] -= q;
    om[2] += q;
    om[46] += q;
    kf = L.kf[114 * kLdsStride];
    kr = kf * ld_uniform(iK, 114);
    q = (kf * C[28]) * C[38] - (kr * C[37]) * C[42];
    om[28] -= q;
    om[38] -= q;
    om[37] += q;
    om[42] += q;
    kf = L.kf[115 * kLdsStride];
    kr = kf * ld_uniform(iK, 115);
    q = (kf * C[38]) * C[45] - (kr * C[33]) * C[33];
    om[38] -= q;
    om[45] -= q;
    om[33] += q;
    om[33] += q;
    kf = L.kf[116 * kLdsStride];
    kr = kf * ld_uniform(iK, 116);
    q = (kf * C[15]) * C[23] - (kr * C[8]) * C[26];
    om[15] -= q;
    om[23] -= q;
    om[8] += q;
    om[26] += q;
    kf = L.kf[117 * kLdsStride];
    kr = kf * ld_uniform(iK, 117);
    q = (kf * C[20]) * C[34] - (kr * C[9]) * C[14];
    om[20] -= q;
    om[34] -= q;
    om[9] += q;
    om[14] += q;
    kf = L.kf[118 * kLdsStride];
    kr = kf * ld_uniform(iK, 118);
    q = (kf * C[20]) * C[23] - (kr * C[13]) * C[13];
    om[20] -= q;
    om[23] -= q;
    om[13] += q;
    om[13] += q;
    kf = L.kf[119 * kLdsStride];
    kr = kf * ld_uniform(iK, 119);
    q = (kf * C[1]) * C[32] - (kr * C[36]) * C[47];
    om[1] -= q;
    om[32] -= q;
    om[36] += q;
    om[47] += q;
    kf = L.kf[120 * kLdsStride];
    kr = kf * ld_uniform(iK, 120);
    q = (kf * C[14]) * C[25] - (kr * C[3]) * C[49];
    om[14] -= q;
    om[25] -= q;
    om[3] += q;
    om[49] += q;
    kf = L.kf[121 * kLdsStride];
    kr = kf * ld_uniform(iK, 121);
    q = (kf * C[23]) * C[33] - (kr * C[29]) * C[48];
    om[23] -= q;
    om[33] -= q;
    om[29] += q;
    om[48] += q;
    kf = L.kf[122 * kLdsStride];
    kr = kf * ld_uniform(iK, 122);
    q = (kf * C[42]) * M - (kr * C[2]) * C[28];
    om[42] -= q;
    om[2] += q;
    om[28] += q;
    kf = L.kf[123 * kLdsStride];
    kr = kf * ld_uniform(iK, 123);
    q = (kf * C[38]) * M - (kr * C[1]) * C[10];
    om[38] -= q;
    om[1] += q;
    om[10] += q;
    kf = L.kf[124 * kLdsStride];
    kr = kf * ld_uniform(iK, 124);
    q = (kf * C[13]) * C[33] - (kr * C[9]) * C[49];
    om[13] -= q;
    om[33] -= q;
    om[9] += q;
    om[49] += q;
    kf = L.kf[125 * kLdsStride];
    kr = kf * ld_uniform(iK, 125);
    q = (kf * C[35]) * C[42] - (kr * C[24]) * C[28];
    om[35] -= q;
    om[42] -= q;
    om[24] += q;
    om[28] += q;
    kf = L.kf[126 * kLdsStride];
    kr = kf * ld_uniform(iK, 126);
    q = (kf * C[2]) * C[21] - (kr * C[3]) * C[36];
    om[2] -= q;
    om[21] -= q;
    om[3] += q;
    om[36] += q;
    kf = L.kf[127 * kLdsStride];
    kr = kf * ld_uniform(iK, 127);
    q = (kf * C[29]) * C[37] - (kr * C[19]) * C[21];
    om[29] -= q;
    om[37] -= q;
    om[19] += q;
    om[21] += q;
    kf = L.kf[128 * kLdsStride];
    kr = kf * ld_uniform(iK, 128);
    q = (kf * C[12]) * C[12] - (kr * C[2]) * C[47];
    om[12] -= q;
    om[12] -= q;
    om[2] += q;
    om[47] += q;
    kf = L.kf[129 * kLdsStride];
    kr = kf * ld_uniform(iK, 129);
    q = (kf * C[19]) * C[31] - (kr * C[25]) * C[35];
    om[19] -= q;
    om[31] -= q;
    om[25] += q;
    om[35] += q;
    kf = L.kf[130 * kLdsStride];
    kr = kf * ld_uniform(iK, 130);
    q = (kf * C[7]) * C[41] - (kr * C[13]) * C[21];
    om[7] -= q;
    om[41] -= q;
    om[13] += q;
    om[21] += q;
    kf = L.kf[131 * kLdsStride];
    kr = kf * ld_uniform(iK, 131);
    q = (kf * C[11]) * C[44] - (kr * C[7]) * C[43];
    om[11] -= q;
    om[44] -= q;
    om[7] += q;
    om[43] += q;
    kf = L.kf[132 * kLdsStride];
    kr = kf * ld_uniform(iK, 132);
    q = (kf * C[2]) * C[26] - (kr * C[14]) * C[23];
    om[2] -= q;
    om[26] -= q;
    om[14] += q;
    om[23] += q;
    kf = L.kf[133 * kLdsStride];
    kr = kf * ld_uniform(iK, 133);
    q = (kf * C[33]) * C[40] - (kr * C[13]) * C[29];
    om[33] -= q;
    om[40] -= q;
    om[13] += q;
    om[29] += q;
    kf = L.kf[134 * kLdsStride];
    kr = kf * ld_uniform(iK, 134);
    q = (kf * C[12]) * C[43] - (kr * C[13]) * C[29];
    om[12] -= q;
    om[43] -= q;
    om[13] += q;
    om[29] += q;
    kf = L.kf[135 * kLdsStride];
    kr = kf * ld_uniform(iK, 135);
    q = (kf * C[9]) * C[16] - (kr * C[8]) * C[13];
    om[9] -= q;
    om[16] -= q;
    om[8] += q;
    om[13] += q;
    kf = L.kf[136 * kLdsStride];
    kr = kf * ld_uniform(iK, 136);
    q = (kf * C[42]) * C[52] - (kr * C[22]) * C[23];
    om[42] -= q;
    om[52] -= q;
    om[22] += q;
    om[23] += q;
    kf = L.kf[137 * kLdsStride];
    kr = kf * ld_uniform(iK, 137);
    q = (kf * C[11]) * C[23] - (kr * C[8]) * C[29];
    om[11] -= q;
    om[23] -= q;
    om[8] += q;
    om[29] += q;
    kf = L.kf[138 * kLdsStride];
    kr = kf * ld_uniform(iK, 138);
    q = (kf * C[5]) * C[48] - (kr * C[1]) * C[15];
    om[5] -= q;
    om[48] -= q;
    om[1] += q;
    om[15] += q;
    kf = L.kf[139 * kLdsStride];
    kr = kf * ld_uniform(iK, 139);
    q = (kf * C[24]) * C[48] - (kr * C[21]) * C[25];
    om[24] -= q;
    om[48] -= q;
    om[21] += q;
    om[25] += q;
    kf = L.kf[140 * kLdsStride];
    kr = kf * ld_uniform(iK, 140);
    q = (kf * C[38]) * C[42] - (kr * C[18]) * C[28];
    om[38] -= q;
    om[42] -= q;
    om[18] += q;
    om[28] += q;
    kf = L.kf[141 * kLdsStride];
    kr = kf * ld_uniform(iK, 141);
    q = (kf * C[30]) * C[45] - (kr * C[31]) * C[52];
    om[30] -= q;
    om[45] -= q;
    om[31] += q;
    om[52] += q;
    kf = L.kf[142 * kLdsStride];
    kr = kf * ld_uniform(iK, 142);
    q = (kf * C[43]) * M - (kr * C[2]) * C[21];
    om[43] -= q;
    om[2] += q;
    om[21] += q;
    kf = L.kf[143 * kLdsStride];
    kr = kf * ld_uniform(iK, 143);
    q = (kf * C[21]) * C[51] - (kr * C[19]) * C[49];
    om[21] -= q;
    om[51] -= q;
    om[19] += q;
    om[49] += q;
    kf = L.kf[144 * kLdsStride];
    kr = kf * ld_uniform(iK, 144);
    q = (kf * C[43]) * C[51] - (kr * C[29]) * C[48];
    om[43] -= q;
    om[51] -= q;
    om[29] += q;
    om[48] += q;
    kf = L.kf[145 * kLdsStride];
    kr = kf * ld_uniform(iK, 145);
    q = (kf * C[26]) * C[46] - (kr * C[30]) * C[37];
    om[26] -= q;
    om[46] -= q;
    om[30] += q;
    om[37] += q;
    kf = L.kf[146 * kLdsStride];
    kr = kf * ld_uniform(iK, 146);
    q = (kf * C[13]) * C[31] - (kr * C[19]) * C[32];
    om[13] -= q;
    om[31] -= q;
    om[19] += q;
    om[32] += q;
    kf = L.kf[147 * kLdsStride];
    kr = kf * ld_uniform(iK, 147);
    q = (kf * C[3]) * C[13] - (kr * C[14]) * C[50];
    om[3] -= q;
    om[13] -= q;
    om[14] += q;
    om[50] += q;
    kf = L.kf[148 * kLdsStride];
    kr = kf * ld_uniform(iK, 148);
    q = (kf * C[26]) * C[28] - (kr * C[8]) * C[41];
    om[26] -= q;
    om[28] -= q;
    om[8] += q;
    om[41] += q;
    kf = L.kf[149 * kLdsStride];
    kr = kf * ld_uniform(iK, 149);
    q = (kf * C[4]) * C[10] - (kr * C[5]) * C[20];
    om[4] -= q;
    om[10] -= q;
    om[5] += q;
    om[20] += q;
    kf = L.kf[150 * kLdsStride];
    kr = kf * ld_uniform(iK, 150);
    q = (kf * C[8]) * C[26] - (kr * C[14]) * C[43];
    om[8] -= q;
    om[26] -= q;
    om[14] += q;
    om[43] += q;
    kf = L.kf[151 * kLdsStride];
    kr = kf * ld_uniform(iK, 151);
    q = (kf * C[9]) * C[49] - (kr * C[16]) * C[48];
    om[9] -= q;
    om[49] -= q;
    om[16] += q;
    om[48] += q;
    kf = L.kf[152 * kLdsStride];
    kr = kf * ld_uniform(iK, 152);
    q = (kf * C[28]) * C[51] - (kr * C[3]) * C[44];
    om[28] -= q;
    om[51] -= q;
    om[3] += q;
    om[44] += q;
    kf = L.kf[153 * kLdsStride];
    kr = kf * ld_uniform(iK, 153);
    q = (kf * C[16]) * C[38] - (kr * C[42]) * C[48];
    om[16] -= q;
    om[38] -= q;
    om[42] += q;
    om[48] += q;
    kf = L.kf[154 * kLdsStride];
    kr = kf * ld_uniform(iK, 154);
    q = (kf * C[7]) * C[24] - (kr * C[11]) * C[48];
    om[7] -= q;
    om[24] -= q;
    om[11] += q;
    om[48] += q;
    kf = L.kf[155 * kLdsStride];
    kr = kf * ld_uniform(iK, 155);
    q = (kf * C[15]) * C[47] - (kr * C[2]) * C[41];
    om[15] -= q;
    om[47] -= q;
    om[2] += q;
    om[41] += q;
    kf = L.kf[156 * kLdsStride];
    kr = kf * ld_uniform(iK, 156);
    q = (kf * C[14]) * C[52] - (kr * C[12]) * C[30];
    om[14] -= q;
    om[52] -= q;
    om[12] += q;
    om[30] += q;
    kf = L.kf[157 * kLdsStride];
    kr = kf * ld_uniform(iK, 157);
    q = (kf * C[8]) * C[9] - (kr * C[28]) * C[50];
    om[8] -= q;
    om[9] -= q;
    om[28] += q;
    om[50] += q;
    kf = L.kf[158 * kLdsStride];
    kr = kf * ld_uniform(iK, 158);
    q = (kf * C[34]) * C[46] - (kr * C[14]) * C[19];
    om[34] -= q;
    om[46] -= q;
    om[14] += q;
    om[19] += q;
    kf = L.kf[159 * kLdsStride];
    kr = kf * ld_uniform(iK, 159);
    q = (kf * C[3]) * C[20] - (kr * C[9]) * C[50];
    om[3] -= q;
    om[20] -= q;
    om[9] += q;
    om[50] += q;
    kf = L.kf[160 * kLdsStride];
    kr = kf * ld_uniform(iK, 160);
    q = (kf * C[20]) * C[45] - (kr * C[25]) * C[37];
    om[20] -= q;
    om[45] -= q;
    om[25] += q;
    om[37] += q;
    kf = L.kf[161 * kLdsStride];
    kr = kf * ld_uniform(iK, 161);
    q = (kf * C[5]) * C[52] - (kr * C[23]) * C[34];
    om[5] -= q;
    om[52] -= q;
    om[23] += q;
    om[34] += q;
    kf = L.kf[162 * kLdsStride];
    kr = kf * ld_uniform(iK, 162);
    q = (kf * C[30]) * M - (kr * C[50]) * C[52];
    om[30] -= q;
    om[50] += q;
    om[52] += q;
    kf = L.kf[163 * kLdsStride];
    kr = kf * ld_uniform(iK, 163);
    q = (kf * C[15]) * C[17] - (kr * C[0]) * C[43];
    om[15] -= q;
    om[17] -= q;
    om[0] += q;
    om[43] += q;
    kf = L.kf[164 * kLdsStride];
    kr = kf * ld_uniform(iK, 164);
    q = (kf * C[8]) * C[47] - (kr * C[2]) * C[35];
    om[8] -= q;
    om[47] -= q;
    om[2] += q;
    om[35] += q;
    kf = L.kf[165 * kLdsStride];
    kr = kf * ld_uniform(iK, 165);
    q = (kf * C[12]) * C[26] - (kr * C[14]) * C[39];
    om[12] -= q;
    om[26] -= q;
    om[14] += q;
    om[39] += q;
    kf = L.kf[166 * kLdsStride];
    kr = kf * ld_uniform(iK, 166);
    q = (kf * C[9]) * C[49] - (kr * C[14]) * C[44];
    om[9] -= q;
    om[49] -= q;
    om[14] += q;
    om[44] += q;
    kf = L.kf[167 * kLdsStride];
    kr = kf * ld_uniform(iK, 167);
    q = (kf * C[8]) * C[42] - (kr * C[11]) * C[28];
    om[8] -= q;
    om[42] -= q;
    om[11] += q;
    om[28] += q;
    kf = L.kf[168 * kLdsStride];
    kr = kf * ld_uniform(iK, 168);
    q = (kf * C[39]) * C[40] - (kr * C[31]) * C[34];
    om[39] -= q;
    om[40] -= q;
    om[31] += q;
    om[34] += q;
    kf = L.kf[169 * kLdsStride];
    kr = kf * ld_uniform(iK, 169);
    q = (kf * C[33]) * C[41] - (kr * C[21]) * C[31];
    om[33] -= q;
    om[41] -= q;
    om[21] += q;
    om[31] += q;
    kf = L.kf[170 * kLdsStride];
    kr = kf * ld_uniform(iK, 170);
    q = (kf * C[9]) * C[39] - (kr * C[18]) * C[47];
    om[9] -= q;
    om[39] -= q;
    om[18] += q;
    om[47] += q;
    kf = L.kf[171 * kLdsStride];
    kr = kf * ld_uniform(iK, 171);
    q = (kf * C[20]) * C[27] - (kr * C[14]) * C[46];
    om[20] -= q;
    om[27] -= q;
    om[14] += q;
    om[46] += q;
    kf = L.kf[172 * kLdsStride];
    kr = kf * ld_uniform(iK, 172);
    q = (kf * C[28]) * C[32] - (kr * C[18]) * C[21];
    om[28] -= q;
    om[32] -= q;
    om[18] += q;
    om[21] += q;
    kf = L.kf[173 * kLdsStride];
    kr = kf * ld_uniform(iK, 173);
    q = (kf * C[12]) * C[20] - (kr * C[7]) * C[19];
    om[12] -= q;
    om[20] -= q;
    om[7] += q;
    om[19] += q;
    kf = L.kf[174 * kLdsStride];
    kr = kf * ld_uniform(iK, 174);
    q = (kf * C[14]) * C[31] - (kr * C[24]) * C[25];
    om[14] -= q;
    om[31] -= q;
    om[24] += q;
    om[25] += q;
    kf = L.kf[175 * kLdsStride];
    kr = kf * ld_uniform(iK, 175);
    q = (kf * C[24]) * C[27] - (kr * C[39]) * C[40];
    om[24] -= q;
    om[27] -= q;
    om[39] += q;
    om[40] += q;
    kf = L.kf[176 * kLdsStride];
    kr = kf * ld_uniform(iK, 176);
    q = (kf * C[16]) * C[51] - (kr * C[12]) * C[33];
    om[16] -= q;
    om[51] -= q;
    om[12] += q;
    om[33] += q;
    kf = L.kf[177 * kLdsStride];
    kr = kf * ld_uniform(iK, 177);
    q = (kf * C[27]) * C[36] - (kr * C[25]) * C[35];
    om[27] -= q;
    om[36] -= q;
    om[25] += q;
    om[35] += q;
    kf = L.kf[178 * kLdsStride];
    kr = kf * ld_uniform(iK, 178);
    q = (kf * C[11]) * C[48] - (kr * C[5]) * C[44];
    om[11] -= q;
    om[48] -= q;
    om[5] += q;
    om[44] += q;
    kf = L.kf[179 * kLdsStride];
    kr = kf * ld_uniform(iK, 179);
    q = (kf * C[1]) * C[24] - (kr * C[19]) * C[23];
    om[1] -= q;
    om[24] -= q;
    om[19] += q;
    om[23] += q;
    kf = L.kf[180 * kLdsStride];
    kr = kf * ld_uniform(iK, 180);
    q = (kf * C[23]) * C[49] - (kr * C[33]) * C[39];
    om[23] -= q;
    om[49] -= q;
    om[33] += q;
    om[39] += q;
    kf = L.kf[181 * kLdsStride];
    kr = kf * ld_uniform(iK, 181);
    q = (kf * C[22]) * C[37] - (kr * C[13]) * C[18];
    om[22] -= q;
    om[37] -= q;
    om[13] += q;
    om[18] += q;
    kf = L.kf[182 * kLdsStride];
    kr = kf * ld_uniform(iK, 182);
    q = (kf * C[13]) * C[33] - (kr * C[10]) * C[45];
    om[13] -= q;
    om[33] -= q;
    om[10] += q;
    om[45] += q;
    kf = L.kf[183 * kLdsStride];
    kr = kf * ld_uniform(iK, 183);
    q = (kf * C[0]) * C[29] - (kr * C[12]) * C[16];
    om[0] -= q;
    om[29] -= q;
    om[12] += q;
    om[16] += q;
    kf = L.kf[184 * kLdsStride];
    kr = kf * ld_uniform(iK, 184);
    q = (kf * C[36]) * C[36] - (kr * C[21]) * C[44];
    om[36] -= q;
    om[36] -= q;
    om[21] += q;
    om[44] += q;
    kf = L.kf[185 * kLdsStride];
    kr = kf * ld_uniform(iK, 185);
    q = (kf * C[3]) * C[7] - (kr * C[0]) * C[4];
    om[3] -= q;
    om[7] -= q;
    om[0] += q;
    om[4] += q;
    kf = L.kf[186 * kLdsStride];
    kr = kf * ld_uniform(iK, 186);
    q = (kf * C[22]) * C[47] - (kr * C[14]) * C[23];
    om[22] -= q;
    om[47] -= q;
    om[14] += q;
    om[23] += q;
    kf = L.kf[187 * kLdsStride];
    kr = kf * ld_uniform(iK, 187);
    q = (kf * C[9]) * C[14] - (kr * C[1]) * C[42];
    om[9] -= q;
    om[14] -= q;
    om[1] += q;
    om[42] += q;
    kf = L.kf[188 * kLdsStride];
    kr = kf * ld_uniform(iK, 188);
    q = (kf * C[9]) * C[38] - (kr * C[16]) * C[20];
    om[9] -= q;
    om[38] -= q;
    om[16] += q;
    om[20] += q;
    kf = L.kf[189 * kLdsStride];
    kr = kf * ld_uniform(iK, 189);
    q = (kf * C[20]) * C[38] - (kr * C[10]) * C[37];
    om[20] -= q;
    om[38] -= q;
    om[10] += q;
    om[37] += q;
    kf = L.kf[190 * kLdsStride];
    kr = kf * ld_uniform(iK, 190);
    q = (kf * C[9]) * C[11] - (kr * C[8]) * C[8];
    om[9] -= q;
    om[11] -= q;
    om[8] += q;
    om[8] += q;
    kf = L.kf[191 * kLdsStride];
    kr = kf * ld_uniform(iK, 191);
    q = (kf * C[6]) * C[38] - (kr * C[10]) * C[34];
    om[6] -= q;
    om[38] -= q;
    om[10] += q;
    om[34] += q;
    kf = L.kf[192 * kLdsStride];
    kr = kf * ld_uniform(iK, 192);
    q = (kf * C[6]) * C[37] - (kr * C[0]) * C[22];
    om[6] -= q;
    om[37] -= q;
    om[0] += q;
    om[22] += q;
    kf = L.kf[193 * kLdsStride];
    kr = kf * ld_uniform(iK, 193);
    q = (kf * C[17]) * C[22] - (kr * C[16]) * C[19];
    om[17] -= q;
    om[22] -= q;
    om[16] += q;
    om[19] += q;
    kf = L.kf[194 * kLdsStride];
    kr = kf * ld_uniform(iK, 194);
    q = (kf * C[28]) * C[51] - (kr * C[14]) * C[46];
    om[28] -= q;
    om[51] -= q;
    om[14] += q;
    om[46] += q;
    kf = L.kf[195 * kLdsStride];
    kr = kf * ld_uniform(iK, 195);
    q = (kf * C[1]) * C[42] - (kr * C[16]) * C[50];
    om[1] -= q;
    om[42] -= q;
    om[16] += q;
    om[50] += q;
    kf = L.kf[196 * kLdsStride];
    kr = kf * ld_uniform(iK, 196);
    q = (kf * C[1]) * C[21] - (kr * C[20]) * C[52];
    om[1] -= q;
    om[21] -= q;
    om[20] += q;
    om[52] += q;
    kf = L.kf[197 * kLdsStride];
    kr = kf * ld_uniform(iK, 197);
    q = (kf * C[8]) * C[44] - (kr * C[20]) * C[35];
    om[8] -= q;
    om[44] -= q;
    om[20] += q;
    om[35] += q;
    kf = L.kf[198 * kLdsStride];
    kr = kf * ld_uniform(iK, 198);
    q = (kf * C[2]) * C[43] - (kr * C[5]) * C[33];
    om[2] -= q;
    om[43] -= q;
    om[5] += q;
    om[33] += q;
    kf = L.kf[199 * kLdsStride];
    kr = kf * ld_uniform(iK, 199);
    q = (kf * C[14]) * C[38] - (kr * C[5]) * C[44];
    om[14] -= q;
    om[38] -= q;
    om[5] += q;
    om[44] += q;
    kf = L.kf[200 * kLdsStride];
    kr = kf * ld_uniform(iK, 200);
    q = (kf * C[7]) * C[15] - (kr * C[11]) * C[37];
    om[7] -= q;
    om[15] -= q;
    om[11] += q;
    om[37] += q;
    kf = L.kf[201 * kLdsStride];
    kr = kf * ld_uniform(iK, 201);
    q = (kf * C[11]) * C[48] - (kr * C[37]) * C[40];
    om[11] -= q;
    om[48] -= q;
    om[37] += q;
    om[40] += q;
    kf = L.kf[202 * kLdsStride];
    kr = kf * ld_uniform(iK, 202);
    q = (kf * C[22]) * C[51] - (kr * C[3]) * C[49];
    om[22] -= q;
    om[51] -= q;
    om[3] += q;
    om[49] += q;
    kf = L.kf[203 * kLdsStride];
    kr = kf * ld_uniform(iK, 203);
    q = (kf * C[48]) * C[50] - (kr * C[0]) * C[33];
    om[48] -= q;
    om[50] -= q;
    om[0] += q;
    om[33] += q;
    kf = L.kf[204 * kLdsStride];
    kr = kf * ld_uniform(iK, 204);
    q = (kf * C[11]) * C[25] - (kr * C[5]) * C[33];
    om[11] -= q;
    om[25] -= q;
    om[5] += q;
    om[33] += q;
    kf = L.kf[205 * kLdsStride];
    kr = kf * ld_uniform(iK, 205);
    q = (kf * C[32]) * C[46] - (kr * C[31]) * C[37];
    om[32] -= q;
    om[46] -= q;
    om[31] += q;
    om[37] += q;
    kf = L.kf[206 * kLdsStride];
    kr = kf * ld_uniform(iK, 206);
    q = (kf * C[19]) * C[33] - (kr * C[12]) * C[36];
    om[19] -= q;
    om[33] -= q;
    om[12] += q;
    om[36] += q;
    kf = L.kf[207 * kLdsStride];
    kr = kf * ld_uniform(iK, 207);
    q = (kf * C[4]) * C[35] - (kr * C[5]) * C[33];
    om[4] -= q;
    om[35] -= q;
    om[5] += q;
    om[33] += q;
    kf = L.kf[208 * kLdsStride];
    kr = kf * ld_uniform(iK, 208);
    q = (kf * C[12]) * C[37] - (kr * C[48]) * C[50];
    om[12] -= q;
    om[37] -= q;
    om[48] += q;
    om[50] += q;
    kf = L.kf[209 * kLdsStride];
    kr = kf * ld_uniform(iK, 209);
    q = (kf * C[10]) * C[47] - (kr * C[0]) * C[35];
    om[10] -= q;
    om[47] -= q;
    om[0] += q;
    om[35] += q;
    kf = L.kf[210 * kLdsStride];
    kr = kf * ld_uniform(iK, 210);
    q = (kf * C[12]) * C[41] - (kr * C[16]) * C[39];
    om[12] -= q;
    om[41] -= q;
    om[16] += q;
    om[39] += q;
    kf = L.kf[211 * kLdsStride];
    kr = kf * ld_uniform(iK, 211);
    q = (kf * C[19]) * C[22] - (kr * C[8]) * C[23];
    om[19] -= q;
    om[22] -= q;
    om[8] += q;
    om[23] += q;
    kf = L.kf[212 * kLdsStride];
    kr = kf * ld_uniform(iK, 212);
    q = (kf * C[14]) * C[22] - (kr * C[16]) * C[40];
    om[14] -= q;
    om[22] -= q;
    om[16] += q;
    om[40] += q;
    kf = L.kf[213 * kLdsStride];
    kr = kf * ld_uniform(iK, 213);
    q = (kf * C[25]) * C[26] - (kr * C[24]) * C[45];
    om[25] -= q;
    om[26] -= q;
    om[24] += q;
    om[45] += q;
    kf = L.kf[214 * kLdsStride];
    kr = kf * ld_uniform(iK, 214);
    q = (kf * C[24]) * C[36] - (kr * C[13]) * C[41];
    om[24] -= q;
    om[36] -= q;
    om[13] += q;
    om[41] += q;
    kf = L.kf[215 * kLdsStride];
    kr = kf * ld_uniform(iK, 215);
    q = (kf * C[12]) * C[46] - (kr * C[33]) * M;
    om[12] -= q;
    om[46] -= q;
    om[33] += q;
    kf = L.kf[216 * kLdsStride];
    kr = kf * ld_uniform(iK, 216);
    q = (kf * C[12]) * C[15] - (kr * C[24]) * C[50];
    om[12] -= q;
    om[15] -= q;
    om[24] += q;
    om[50] += q;
    kf = L.kf[217 * kLdsStride];
    kr = kf * ld_uniform(iK, 217);
    q = (kf * C[13]) * C[49] - (kr * C[31]) * C[46];
    om[13] -= q;
    om[49] -= q;
    om[31] += q;
    om[46] += q;
    kf = L.kf[218 * kLdsStride];
    kr = kf * ld_uniform(iK, 218);
    q = (kf * C[1]) * C[5] - (kr * C[3]) * C[19];
    om[1] -= q;
    om[5] -= q;
    om[3] += q;
    om[19] += q;
    kf = L.kf[219 * kLdsStride];
    kr = kf * ld_uniform(iK, 219);
    q = (kf * C[13]) * C[52] - (kr * C[24]) * C[51];
    om[13] -= q;
    om[52] -= q;
    om[24] += q;
    om[51] += q;
    kf = L.kf[220 * kLdsStride];
    kr = kf * ld_uniform(iK, 220);
    q = (kf * C[4]) * C[27] - (kr * C[5]) * C[47];
    om[4] -= q;
    om[27] -= q;
    om[5] += q;
    om[47] += q;
    kf = L.kf[221 * kLdsStride];
    kr = kf * ld_uniform(iK, 221);
    q = (kf * C[19]) * C[19] - (kr * C[1]) * C[16];
    om[19] -= q;
    om[19] -= q;
    om[1] += q;
    om[16] += q;
    kf = L.kf[222 * kLdsStride];
    kr = kf * ld_uniform(iK, 222);
    q = (kf * C[0]) * C[16] - (kr * C[2]) * C[38];
    om[0] -= q;
    om[16] -= q;
    om[2] += q;
    om[38] += q;
    kf = L.kf[223 * kLdsStride];
    kr = kf * ld_uniform(iK, 223);
    q = (kf * C[30]) * C[37] - (kr * C[33]) * C[35];
    om[30] -= q;
    om[37] -= q;
    om[33] += q;
    om[35] += q;
    kf = L.kf[224 * kLdsStride];
    kr = kf * ld_uniform(iK, 224);
    q = (kf * C[9]) * C[49] - (kr * C[0]) * C[32];
    om[9] -= q;
    om[49] -= q;
    om[0] += q;
    om[32] += q;
    kf = L.kf[225 * kLdsStride];
    kr = kf * ld_uniform(iK, 225);
    q = (kf * C[20]) * C[33] - (kr * C[13]) * C[37];
    om[20] -= q;
    om[33] -= q;
    om[13] += q;
    om[37] += q;
    kf = L.kf[226 * kLdsStride];
    kr = kf * ld_uniform(iK, 226);
    q = (kf * C[14]) * C[18] - (kr * C[13]) * C[22];
    om[14] -= q;
    om[18] -= q;
    om[13] += q;
    om[22] += q;
    kf = L.kf[227 * kLdsStride];
    kr = kf * ld_uniform(iK, 227);
    q = (kf * C[14]) * C[27] - (kr * C[3]) * C[39];
    om[14] -= q;
    om[27] -= q;
    om[3] += q;
    om[39] += q;
    kf = L.kf[228 * kLdsStride];
    kr = kf * ld_uniform(iK, 228);
    q = (kf * C[14]) * C[19] - (kr * C[11]) * C[51];
    om[14] -= q;
    om[19] -= q;
    om[11] += q;
    om[51] += q;
    kf = L.kf[229 * kLdsStride];
    kr = kf * ld_uniform(iK, 229);
    q = (kf * C[24]) * C[42] - (kr * C[11]) * C[43];
    om[24] -= q;
    om[42] -= q;
    om[11] += q;
    om[43] += q;
    kf = L.kf[230 * kLdsStride];
    kr = kf * ld_uniform(iK, 230);
    q = (kf * C[7]) * C[27] - (kr * C[9]) * C[47];
    om[7] -= q;
    om[27] -= q;
    om[9] += q;
    om[47] += q;
    kf = L.kf[231 * kLdsStride];
    kr = kf * ld_uniform(iK, 231);
    q = (kf * C[31]) * M - (kr * C[45]) * C[50];
    om[31] -= q;
    om[45] += q;
    om[50] += q;
    kf = L.kf[232 * kLdsStride];
    kr = kf * ld_uniform(iK, 232);
    q = (kf * C[27]) * C[42] - (kr * C[4]) * C[24];
    om[27] -= q;
    om[42] -= q;
    om[4] += q;
    om[24] += q;
    kf = L.kf[233 * kLdsStride];
    kr = kf * ld_uniform(iK, 233);
    q = (kf * C[20]) * C[52] - (kr * C[23]) * C[46];
    om[20] -= q;
    om[52] -= q;
    om[23] += q;
    om[46] += q;
    kf = L.kf[234 * kLdsStride];
    kr = kf * ld_uniform(iK, 234);
    q = (kf * C[27]) * C[33] - (kr * C[19]) * C[39];
    om[27] -= q;
    om[33] -= q;
    om[19] += q;
    om[39] += q;
    kf = L.kf[235 * kLdsStride];
    kr = kf * ld_uniform(iK, 235);
    q = (kf * C[1]) * C[35] - (kr * C[31]) * M;
    om[1] -= q;
    om[35] -= q;
    om[31] += q;
    kf = L.kf[236 * kLdsStride];
    kr = kf * ld_uniform(iK, 236);
    q = (kf * C[14]) * C[30] - (kr * C[22]) * C[52];
    om[14] -= q;
    om[30] -= q;
    om[22] += q;
    om[52] += q;
    kf = L.kf[237 * kLdsStride];
    kr = kf * ld_uniform(iK, 237);
    q = (kf * C[6]) * C[16] - (kr * C[8]) * C[34];
    om[6] -= q;
    om[16] -= q;
    om[8] += q;
    om[34] += q;
    kf = L.kf[238 * kLdsStride];
    kr = kf * ld_uniform(iK, 238);
    q = (kf * C[40]) * C[51] - (kr * C[1]) * C[29];
    om[40] -= q;
    om[51] -= q;
    om[1] += q;
    om[29] += q;
    kf = L.kf[239 * kLdsStride];
    kr = kf * ld_uniform(iK, 239);
    q = (kf * C[4]) * C[22] - (kr * C[28]) * C[34];
    om[4] -= q;
    om[22] -= q;
    om[28] += q;
    om[34] += q;
    kf = L.kf[240 * kLdsStride];
    kr = kf * ld_uniform(iK, 240);
    q = (kf * C[12]) * C[43] - (kr * C[15]) * C[47];
    om[12] -= q;
    om[43] -= q;
    om[15] += q;
    om[47] += q;
    kf = L.kf[241 * kLdsStride];
    kr = kf * ld_uniform(iK, 241);
    q = (kf * C[18]) * C[39] - (kr * C[30]) * C[38];
    om[18] -= q;
    om[39] -= q;
    om[30] += q;
    om[38] += q;
    kf = L.kf[242 * kLdsStride];
    kr = kf * ld_uniform(iK, 242);
    q = (kf * C[10]) * C[31] - (kr * C[15]) * C[48];
    om[10] -= q;
    om[31] -= q;
    om[15] += q;
    om[48] += q;
    kf = L.kf[243 * kLdsStride];
    kr = kf * ld_uniform(iK, 243);
    q = (kf * C[19]) * C[32] - (kr * C[33]) * C[35];
    om[19] -= q;
    om[32] -= q;
    om[33] += q;
    om[35] += q;
    kf = L.kf[244 * kLdsStride];
    kr = kf * ld_uniform(iK, 244);
    q = (kf * C[23]) * C[25] - (kr * C[13]) * C[52];
    om[23] -= q;
    om[25] -= q;
    om[13] += q;
    om[52] += q;
    kf = L.kf[245 * kLdsStride];
    kr = kf * ld_uniform(iK, 245);
    q = (kf * C[15]) * C[51] - (kr * C[41]) * M;
    om[15] -= q;
    om[51] -= q;
    om[41] += q;
    kf = L.kf[246 * kLdsStride];
    kr = kf * ld_uniform(iK, 246);
    q = (kf * C[4]) * C[23] - (kr * C[3]) * C[35];
    om[4] -= q;
    om[23] -= q;
    om[3] += q;
    om[35] += q;
    kf = L.kf[247 * kLdsStride];
    kr = kf * ld_uniform(iK, 247);
    q = (kf * C[10]) * C[51] - (kr * C[48]) * C[50];
    om[10] -= q;
    om[51] -= q;
    om[48] += q;
    om[50] += q;
    kf = L.kf[248 * kLdsStride];
    kr = kf * ld_uniform(iK, 248);
    q = (kf * C[5]) * C[48] - (kr * C[4]) * C[33];
    om[5] -= q;
    om[48] -= q;
    om[4] += q;
    om[33] += q;
    kf = L.kf[249 * kLdsStride];
    kr = kf * ld_uniform(iK, 249);
    q = (kf * C[11]) * C[33] - (kr * C[16]) * C[16];
    om[11] -= q;
    om[33] -= q;
    om[16] += q;
    om[16] += q;
    kf = L.kf[250 * kLdsStride];
    kr = kf * ld_uniform(iK, 250);
    q = (kf * C[10]) * C[39] - (kr * C[13]) * C[35];
    om[10] -= q;
    om[39] -= q;
    om[13] += q;
    om[35] += q;
    kf = L.kf[251 * kLdsStride];
    kr = kf * ld_uniform(iK, 251);
    q = (kf * C[19]) * C[45] - (kr * C[1]) * C[31];
    om[19] -= q;
    om[45] -= q;
    om[1] += q;
    om[31] += q;
    kf = L.kf[252 * kLdsStride];
    kr = kf * ld_uniform(iK, 252);
    q = (kf * C[10]) * C[30] - (kr * C[18]) * C[23];
    om[10] -= q;
    om[30] -= q;
    om[18] += q;
    om[23] += q;
    kf = L.kf[253 * kLdsStride];
    kr = kf * ld_uniform(iK, 253);
    q = (kf * C[19]) * C[35] - (kr * C[27]) * C[38];
    om[19] -= q;
    om[35] -= q;
    om[27] += q;
    om[38] += q;
    kf = L.kf[254 * kLdsStride];
    kr = kf * ld_uniform(iK, 254);
    q = (kf * C[12]) * C[43] - (kr * C[19]) * C[24];
    om[12] -= q;
    om[43] -= q;
    om[19] += q;
    om[24] += q;
    kf = L.kf[255 * kLdsStride];
    kr = kf * ld_uniform(iK, 255);
    q = (kf * C[8]) * C[43] - (kr * C[24]) * C[28];
    om[8] -= q;
    om[43] -= q;
    om[24] += q;
    om[28] += q;
    kf = L.kf[256 * kLdsStride];
    kr = kf * ld_uniform(iK, 256);
    q = (kf * C[20]) * C[23] - (kr * C[7]) * C[35];
    om[20] -= q;
    om[23] -= q;
    om[7] += q;
    om[35] += q;
    kf = L.kf[257 * kLdsStride];
    kr = kf * ld_uniform(iK, 257);
    q = (kf * C[17]) * C[36] - (kr * C[19]) * C[44];
    om[17] -= q;
    om[36] -= q;
    om[19] += q;
    om[44] += q;
    kf = L.kf[258 * kLdsStride];
    kr = kf * ld_uniform(iK, 258);
    q = (kf * C[11]) * C[21] - (kr * C[8]) * C[43];
    om[11] -= q;
    om[21] -= q;
    om[8] += q;
    om[43] += q;
    kf = L.kf[259 * kLdsStride];
    kr = kf * ld_uniform(iK, 259);
    q = (kf * C[15]) * C[17] - (kr * C[25]) * C[28];
    om[15] -= q;
    om[17] -= q;
    om[25] += q;
    om[28] += q;
    kf = L.kf[260 * kLdsStride];
    kr = kf * ld_uniform(iK, 260);
    q = (kf * C[29]) * C[31] - (kr * C[43]) * C[52];
    om[29] -= q;
    om[31] -= q;
    om[43] += q;
    om[52] += q;
    kf = L.kf[261 * kLdsStride];
    kr = kf * ld_uniform(iK, 261);
    q = (kf * C[12]) * C[25] - (kr * C[1]) * C[23];
    om[12] -= q;
    om[25] -= q;
    om[1] += q;
    om[23] += q;
    kf = L.kf[262 * kLdsStride];
    kr = kf * ld_uniform(iK, 262);
    q = (kf * C[21]) * C[45] - (kr * C[36]) * C[39];
    om[21] -= q;
    om[45] -= q;
    om[36] += q;
    om[39] += q;
    kf = L.kf[263 * kLdsStride];
    kr = kf * ld_uniform(iK, 263);
    q = (kf * C[24]) * C[25] - (kr * C[13]) * C[30];
    om[24] -= q;
    om[25] -= q;
    om[13] += q;
    om[30] += q;
    kf = L.kf[264 * kLdsStride];
    kr = kf * ld_uniform(iK, 264);
    q = (kf * C[22]) * C[52] - (kr * C[31]) * C[34];
    om[22] -= q;
    om[52] -= q;
    om[31] += q;
    om[34] += q;
    kf = L.kf[265 * kLdsStride];
    kr = kf * ld_uniform(iK, 265);
    q = (kf * C[12]) * C[14] - (kr * C[27]) * C[50];
    om[12] -= q;
    om[14] -= q;
    om[27] += q;
    om[50] += q;
    kf = L.kf[266 * kLdsStride];
    kr = kf * ld_uniform(iK, 266);
    q = (kf * C[23]) * C[24] - (kr * C[15]) * C[52];
    om[23] -= q;
    om[24] -= q;
    om[15] += q;
    om[52] += q;
    kf = L.kf[267 * kLdsStride];
    kr = kf * ld_uniform(iK, 267);
    q = (kf * C[26]) * C[50] - (kr * C[22]) * C[25];
    om[26] -= q;
    om[50] -= q;
    om[22] += q;
    om[25] += q;
    kf = L.kf[268 * kLdsStride];
    kr = kf * ld_uniform(iK, 268);
    q = (kf * C[18]) * C[50] - (kr * C[4]) * C[38];
    om[18] -= q;
    om[50] -= q;
    om[4] += q;
    om[38] += q;
    kf = L.kf[269 * kLdsStride];
    kr = kf * ld_uniform(iK, 269);
    q = (kf * C[19]) * C[23] - (kr * C[0]) * C[30];
    om[19] -= q;
    om[23] -= q;
    om[0] += q;
    om[30] += q;
    kf = L.kf[270 * kLdsStride];
    kr = kf * ld_uniform(iK, 270);
    q = (kf * C[9]) * C[45] - (kr * C[18]) * C[51];
    om[9] -= q;
    om[45] -= q;
    om[18] += q;
    om[51] += q;
    kf = L.kf[271 * kLdsStride];
    kr = kf * ld_uniform(iK, 271);
    q = (kf * C[17]) * C[18] - (kr * C[10]) * C[25];
    om[17] -= q;
    om[18] -= q;
    om[10] += q;
    om[25] += q;
    kf = L.kf[272 * kLdsStride];
    kr = kf * ld_uniform(iK, 272);
    q = (kf * C[19]) * C[41] - (kr * C[16]) * C[31];
    om[19] -= q;
    om[41] -= q;
    om[16] += q;
    om[31] += q;
    kf = L.kf[273 * kLdsStride];
    kr = kf * ld_uniform(iK, 273);
    q = (kf * C[13]) * C[25] - (kr * C[20]) * C[52];
    om[13] -= q;
    om[25] -= q;
    om[20] += q;
    om[52] += q;
    kf = L.kf[274 * kLdsStride];
    kr = kf * ld_uniform(iK, 274);
    q = (kf * C[40]) * C[43] - (kr * C[22]) * C[24];
    om[40] -= q;
    om[43] -= q;
    om[22] += q;
    om[24] += q;
    kf = L.kf[275 * kLdsStride];
    kr = kf * ld_uniform(iK, 275);
    q = (kf * C[29]) * C[37] - (kr * C[32]) * C[50];
    om[29] -= q;
    om[37] -= q;
    om[32] += q;
    om[50] += q;
    kf = L.kf[276 * kLdsStride];
    kr = kf * ld_uniform(iK, 276);
    q = (kf * C[2]) * C[46] - (kr * C[13]) * M;
    om[2] -= q;
    om[46] -= q;
    om[13] += q;
    kf = L.kf[277 * kLdsStride];
    kr = kf * ld_uniform(iK, 277);
    q = (kf * C[1]) * C[11] - (kr * C[0]) * C[40];
    om[1] -= q;
    om[11] -= q;
    om[0] += q;
    om[40] += q;
    kf = L.kf[278 * kLdsStride];
    kr = kf * ld_uniform(iK, 278);
    q = (kf * C[27]) * C[44] - (kr * C[37]) * C[52];
    om[27] -= q;
    om[44] -= q;
    om[37] += q;
    om[52] += q;
    kf = L.kf[279 * kLdsStride];
    kr = kf * ld_uniform(iK, 279);
    q = (kf * C[18]) * C[29] - (kr * C[39]) * C[42];
    om[18] -= q;
    om[29] -= q;
    om[39] += q;
    om[42] += q;
    kf = L.kf[280 * kLdsStride];
    kr = kf * ld_uniform(iK, 280);
    q = (kf * C[9]) * C[17] - (kr * C[0]) * C[13];
    om[9] -= q;
    om[17] -= q;
    om[0] += q;
    om[13] += q;
    kf = L.kf[281 * kLdsStride];
    kr = kf * ld_uniform(iK, 281);
    q = (kf * C[19]) * C[20] - (kr * C[10]) * C[17];
    om[19] -= q;
    om[20] -= q;
    om[10] += q;
    om[17] += q;
    kf = L.kf[282 * kLdsStride];
    kr = kf * ld_uniform(iK, 282);
    q = (kf * C[33]) * C[35] - (kr * C[38]) * C[39];
    om[33] -= q;
    om[35] -= q;
    om[38] += q;
    om[39] += q;
    kf = L.kf[283 * kLdsStride];
    kr = kf * ld_uniform(iK, 283);
    q = (kf * C[40]) * C[48] - (kr * C[1]) * C[43];
    om[40] -= q;
    om[48] -= q;
    om[1] += q;
    om[43] += q;
    kf = L.kf[284 * kLdsStride];
    kr = kf * ld_uniform(iK, 284);
    q = (kf * C[8]) * C[29] - (kr * C[14]) * C[22];
    om[8] -= q;
    om[29] -= q;
    om[14] += q;
    om[22] += q;
    kf = L.kf[285 * kLdsStride];
    kr = kf * ld_uniform(iK, 285);
    q = (kf * C[7]) * C[32] - (kr * C[35]) * C[37];
    om[7] -= q;
    om[32] -= q;
    om[35] += q;
    om[37] += q;
    kf = L.kf[286 * kLdsStride];
    kr = kf * ld_uniform(iK, 286);
    q = (kf * C[17]) * C[27] - (kr * C[0]) * C[52];
    om[17] -= q;
    om[27] -= q;
    om[0] += q;
    om[52] += q;
    kf = L.kf[287 * kLdsStride];
    kr = kf * ld_uniform(iK, 287);
    q = (kf * C[19]) * C[49] - (kr * C[37]) * C[52];
    om[19] -= q;
    om[49] -= q;
    om[37] += q;
    om[52] += q;
    kf = L.kf[288 * kLdsStride];
    kr = kf * ld_uniform(iK, 288);
    q = (kf * C[1]) * C[11] - (kr * C[22]) * M;
    om[1] -= q;
    om[11] -= q;
    om[22] += q;
    kf = L.kf[289 * kLdsStride];
    kr = kf * ld_uniform(iK, 289);
    q = (kf * C[27]) * C[36] - (kr * C[23]) * C[33];
    om[27] -= q;
    om[36] -= q;
    om[23] += q;
    om[33] += q;
    kf = L.kf[290 * kLdsStride];
    kr = kf * ld_uniform(iK, 290);
    q = (kf * C[36]) * C[52] - (kr * C[35]) * C[45];
    om[36] -= q;
    om[52] -= q;
    om[35] += q;
    om[45] += q;
    kf = L.kf[291 * kLdsStride];
    kr = kf * ld_uniform(iK, 291);
    q = (kf * C[17]) * C[21] - (kr * C[20]) * C[39];
    om[17] -= q;
    om[21] -= q;
    om[20] += q;
    om[39] += q;
    kf = L.kf[292 * kLdsStride];
    kr = kf * ld_uniform(iK, 292);
    q = (kf * C[22]) * C[48] - (kr * C[24]) * C[46];
    om[22] -= q;
    om[48] -= q;
    om[24] += q;
    om[46] += q;
    kf = L.kf[293 * kLdsStride];
    kr = kf * ld_uniform(iK, 293);
    q = (kf * C[11]) * C[27] - (kr * C[6]) * C[35];
    om[11] -= q;
    om[27] -= q;
    om[6] += q;
    om[35] += q;
    kf = L.kf[294 * kLdsStride];
    kr = kf * ld_uniform(iK, 294);
    q = (kf * C[33]) * C[33] - (kr * C[25]) * C[36];
    om[33] -= q;
    om[33] -= q;
    om[25] += q;
    om[36] += q;
    kf = L.kf[295 * kLdsStride];
    kr = kf * ld_uniform(iK, 295);
    q = (kf * C[8]) * C[12] - (kr * C[22]) * M;
    om[8] -= q;
    om[12] -= q;
    om[22] += q;
    kf = L.kf[296 * kLdsStride];
    kr = kf * ld_uniform(iK, 296);
    q = (kf * C[29]) * C[33] - (kr * C[13]) * C[30];
    om[29] -= q;
    om[33] -= q;
    om[13] += q;
    om[30] += q;
    kf = L.kf[297 * kLdsStride];
    kr = kf * ld_uniform(iK, 297);
    q = (kf * C[23]) * C[52] - (kr * C[30]) * C[47];
    om[23] -= q;
    om[52] -= q;
    om[30] += q;
    om[47] += q;
    kf = L.kf[298 * kLdsStride];
    kr = kf * ld_uniform(iK, 298);
    q = (kf * C[0]) * C[22] - (kr * C[11]) * C[17];
    om[0] -= q;
    om[22] -= q;
    om[11] += q;
    om[17] += q;
    kf = L.kf[299 * kLdsStride];
    kr = kf * ld_uniform(iK, 299);
    q = (kf * C[34]) * C[43] - (kr * C[11]) * C[30];
    om[34] -= q;
    om[43] -= q;
    om[11] += q;
    om[30] += q;
    kf = L.kf[300 * kLdsStride];
    kr = kf * ld_uniform(iK, 300);
    q = (kf * C[15]) * C[47] - (kr * C[18]) * C[27];
    om[15] -= q;
    om[47] -= q;
    om[18] += q;
    om[27] += q;
    kf = L.kf[301 * kLdsStride];
    kr = kf * ld_uniform(iK, 301);
    q = (kf * C[25]) * C[50] - (kr * C[9]) * C[47];
    om[25] -= q;
    om[50] -= q;
    om[9] += q;
    om[47] += q;
    kf = L.kf[302 * kLdsStride];
    kr = kf * ld_uniform(iK, 302);
    q = (kf * C[35]) * C[43] - (kr * C[18]) * C[26];
    om[35] -= q;
    om[43] -= q;
    om[18] += q;
    om[26] += q;
    kf = L.kf[303 * kLdsStride];
    kr = kf * ld_uniform(iK, 303);
    q = (kf * C[8]) * C[19] - (kr * C[2]) * C[18];
    om[8] -= q;
    om[19] -= q;
    om[2] += q;
    om[18] += q;
    kf = L.kf[304 * kLdsStride];
    kr = kf * ld_uniform(iK, 304);
    q = (kf * C[34]) * C[38] - (kr * C[3]) * C[21];
    om[34] -= q;
    om[38] -= q;
    om[3] += q;
    om[21] += q;
    kf = L.kf[305 * kLdsStride];
    kr = kf * ld_uniform(iK, 305);
    q = (kf * C[5]) * C[24] - (kr * C[22]) * C[40];
    om[5] -= q;
    om[24] -= q;
    om[22] += q;
    om[40] += q;
    kf = L.kf[306 * kLdsStride];
    kr = kf * ld_uniform(iK, 306);
    q = (kf * C[1]) * C[4] - (kr * C[3]) * C[17];
    om[1] -= q;
    om[4] -= q;
    om[3] += q;
    om[17] += q;
    kf = L.kf[307 * kLdsStride];
    kr = kf * ld_uniform(iK, 307);
    q = (kf * C[23]) * C[38] - (kr * C[8]) * C[49];
    om[23] -= q;
    om[38] -= q;
    om[8] += q;
    om[49] += q;
    kf = L.kf[308 * kLdsStride];
    kr = kf * ld_uniform(iK, 308);
    q = (kf * C[37]) * C[52] - (kr * C[21]) * C[51];
    om[37] -= q;
    om[52] -= q;
    om[21] += q;
    om[51] += q;
    kf = L.kf[309 * kLdsStride];
    kr = kf * ld_uniform(iK, 309);
    q = (kf * C[35]) * C[46] - (kr * C[20]) * C[39];
    om[35] -= q;
    om[46] -= q;
    om[20] += q;
    om[39] += q;
    kf = L.kf[310 * kLdsStride];
    kr = kf * ld_uniform(iK, 310);
    q = (kf * C[31]) * C[42] - (kr * C[8]) * C[41];
    om[31] -= q;
    om[42] -= q;
    om[8] += q;
    om[41] += q;
    kf = L.kf[311 * kLdsStride];
    kr = kf * ld_uniform(iK, 311);
    q = (kf * C[25]) * C[36] - (kr * C[38]) * C[45];
    om[25] -= q;
    om[36] -= q;
    om[38] += q;
    om[45] += q;
    kf = L.kf[312 * kLdsStride];
    kr = kf * ld_uniform(iK, 312);
    q = (kf * C[29]) * C[32] - (kr * C[24]) * C[31];
    om[29] -= q;
    om[32] -= q;
    om[24] += q;
    om[31] += q;
    kf = L.kf[313 * kLdsStride];
    kr = kf * ld_uniform(iK, 313);
    q = (kf * C[14]) * C[37] - (kr * C[36]) * C[50];
    om[14] -= q;
    om[37] -= q;
    om[36] += q;
    om[50] += q;
    kf = L.kf[314 * kLdsStride];
    kr = kf * ld_uniform(iK, 314);
    q = (kf * C[2]) * C[22] - (kr * C[3]) * C[16];
    om[2] -= q;
    om[22] -= q;
    om[3] += q;
    om[16] += q;
    kf = L.kf[315 * kLdsStride];
    kr = kf * ld_uniform(iK, 315);
    q = (kf * C[15]) * C[46] - (kr * C[13]) * C[18];
    om[15] -= q;
    om[46] -= q;
    om[13] += q;
    om[18] += q;
    kf = L.kf[316 * kLdsStride];
    kr = kf * ld_uniform(iK, 316);
    q = (kf * C[15]) * C[38] - (kr * C[36]) * C[42];
    om[15] -= q;
    om[38] -= q;
    om[36] += q;
    om[42] += q;
    kf = L.kf[317 * kLdsStride];
    kr = kf * ld_uniform(iK, 317);
    q = (kf * C[16]) * C[30] - (kr * C[31]) * C[40];
    om[16] -= q;
    om[30] -= q;
    om[31] += q;
    om[40] += q;
    kf = L.kf[318 * kLdsStride];
    kr = kf * ld_uniform(iK, 318);
    q = (kf * C[25]) * C[43] - (kr * C[24]) * C[33];
    om[25] -= q;
    om[43] -= q;
    om[24] += q;
    om[33] += q;
    kf = L.kf[319 * kLdsStride];
    kr = kf * ld_uniform(iK, 319);
    q = (kf * C[8]) * C[51] - (kr * C[25]) * C[50];
    om[8] -= q;
    om[51] -= q;
    om[25] += q;
    om[50] += q;
    kf = L.kf[320 * kLdsStride];
    kr = kf * ld_uniform(iK, 320);
    q = (kf * C[11]) * C[27] - (kr * C[3]) * C[24];
    om[11] -= q;
    om[27] -= q;
    om[3] += q;
    om[24] += q;
    kf = L.kf[321 * kLdsStride];
    kr = kf * ld_uniform(iK, 321);
    q = (kf * C[18]) * C[45] - (kr * C[26]) * C[46];
    om[18] -= q;
    om[45] -= q;
    om[26] += q;
    om[46] += q;
    kf = L.kf[322 * kLdsStride];
    kr = kf * ld_uniform(iK, 322);
    q = (kf * C[22]) * M - (kr * C[0]) * C[40];
    om[22] -= q;
    om[0] += q;
    om[40] += q;
    kf = L.kf[323 * kLdsStride];
    kr = kf * ld_uniform(iK, 323);
    q = (kf * C[2]) * C[5] - (kr * C[6]) * C[50];
    om[2] -= q;
    om[5] -= q;
    om[6] += q;
    om[50] += q;
    kf = L.kf[324 * kLdsStride];
    kr = kf * ld_uniform(iK, 324);
    q = (kf * C[28]) * C[52] - (kr * C[5]) * C[49];
    om[28] -= q;
    om[52] -= q;
    om[5] += q;
    om[49] += q;
#pragma unroll
    for (int k = 0; k < N; ++k) f[k] = (ld_uniform(W, k) * om[k]) * L.irho;
  }
};

// Group variant: 32 lanes per system (rk_group.hpp).
struct GNet {
  static constexpr int N = 53;
  static constexpr int NR = 325;
  static constexpr int kL = 32;
  static constexpr int kGroupLanes = 32;
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  // RKCK: three waves per SIMD, its loop fits 168 registers but for a few spills
  // outside the evaluations (53 species, 65536 systems, in one session: three waves
  // 636 ms, two 698)
  static constexpr int kWavesPerEuRkc = 2;
  static constexpr int kWavesPerEuRkck = 3;
  static constexpr int S = 2;
  static constexpr int R = 11;
  static constexpr int kMSlot = 10;   // first slot that may hold a [M] reaction
  static constexpr int kOffC = 0;
  static constexpr int kOffQ = 54;
  static constexpr int kSentinel = 352;
  static constexpr int kNegOff = 407;
  static constexpr int kOffRed = 408;
  static constexpr int kLdsPerSystem = 814;
  static constexpr int kTermLen = 48;
  static constexpr int kChunk = 4;
  using Params = const double*;
  static constexpr int kSp[64] = {
      -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, 6, 50, 18, 22, 35,
      12, 27, 37, 11, 20, 49, 17, 36, 51, 47, 21, 4, 38, 46, 48, 2,
      33, 13, 14, 19, 23, 16, 8, 25, 9, 52, 31, 24, 44, 41, 26, 32,
      42, 30, 29, 34, 10, 43, 1, 15, 39, 0, 3, 28, 45, 40, 7, 5};
  static constexpr int16_t kRxOf[352] = {
      118, 133, 266, 61, 63, 264, 113, 22, 153, 315, 250, 30, 311, 312, 309, 67,
      132, 192, 252, 319, 283, 13, 121, 3, 225, 172, 219, 188, 248, 205, 155, 70,
      157, 217, 28, 21, 110, 64, 226, 202, 136, 115, 42, 147, 218, 98, 95, -1,
      62, -1, 170, 7, 137, 269, 15, 185, 107, 233, 168, 46, 129, 73, 320, 127,
      48, 291, 105, 221, 68, 220, 154, 169, 232, 249, 83, 175, 224, 65, 214, 197,
      138, 39, 161, 324, 44, 279, 227, 321, 33, 265, 34, 194, 198, 281, 165, 189,
      26, 93, 146, 102, 243, 313, 228, 109, 37, 271, 32, 167, 230, 284, 278, 256,
      45, 280, 180, 114, 158, 77, 179, 181, 277, 285, 212, -1, 209, 43, 318, -1,
      71, 177, -1, 14, 274, 246, 263, 190, 208, 69, 196, 81, 222, 156, 191, 120,
      52, 199, 270, 302, 84, 54, 171, 124, 108, 160, 206, 216, 51, 111, -1, 40,
      240, 184, 86, 2, 173, 268, 16, 75, 159, 139, 78, 50, 282, 101, 4, 27,
      174, -1, 97, 260, 47, 314, 128, 100, 85, 89, 244, 134, 18, 82, 1, 57,
      262, 35, 308, 251, 91, 90, 261, 23, 301, 58, -1, -1, 238, 72, 141, 131,
      126, 257, 56, 106, 292, 213, 59, 323, 103, 79, 29, 203, 140, 293, 287, 242,
      306, 317, 204, 223, 183, -1, 66, 290, 5, 38, 116, 17, 247, 12, 20, 234,
      200, -1, 304, 125, 286, 88, 275, 36, 53, 255, 210, 201, 195, 178, 187, 258,
      -1, 9, 303, 150, 254, 298, 74, 151, 305, 144, 297, 87, 55, 149, 193, 76,
      272, 164, 41, 96, 10, 237, 135, 241, 166, 24, 207, 267, 49, 259, 94, 119,
      130, 307, 299, 99, 31, 19, 6, 229, 148, 0, 112, 163, 296, 117, 253, 239,
      310, 152, 211, 143, 176, 11, 273, 186, 60, 289, 182, 316, 145, 294, 236, 300,
      8, 25, -1, -1, 80, -1, 162, -1, -1, -1, 104, 322, -1, 215, -1, 231,
      -1, -1, -1, -1, -1, 122, 235, 245, -1, -1, 142, 276, 288, 295, 92, 123};
  // each lane's LDS offsets (in units of 2^kAddrShift bytes) in the wave's areas,
  // two to a word, contiguous and 16-byte aligned (read as whole vectors at every
  // evaluation): the rates' operands, the terms
  static constexpr int kAddrShift = 0;
  static constexpr int kOpWords = 24;
  static constexpr int kTmWords = 24;
  alignas(16) static constexpr uint32_t kOp[1536] = {
      12058784, 6815848, 4718656, 26214624, 26214424, 3145728, 22544384, 8388712, 25166144, 20447304, 22544480, 24641656, 23593128, 20447520, 2097160, 8912920,
      0, 0, 21495864, 11010152, 27787408, 7340088, 0, 0, 20971784, 15204456, 25690216, 24117496, 11010184, 20447392, 27263264, 20447496,
      18874584, 18350280, 18874656, 23068840, 16252960, 22544480, 15728768, 20971768, 12583040, 16253016, 19923128, 25690176, 13107216, 27787448, 0, 0,
      12583096, 27263096, 12058728, 23068944, 25690144, 17301616, 16253032, 16777368, 0, 0, 18350280, 23593088, 27263272, 26738856, 13107288, 17301544,
      9961536, 9437200, 22544656, 15728728, 0, 0, 0, 0, 23593008, 24641856, 6291544, 9961512, 9961624, 8388616, 20971736, 17825976,
      6815848, 18350136, 23593032, 17301656, 23593112, 16252936, 19398896, 18350344, 13631552, 22544496, 14155808, 20971616, 0, 0, 0, 0,
      13631488, 25690144, 25165896, 13107360, 27263032, 26738816, 16777368, 18350344, 22544704, 12583088, 10485856, 9961528, 26738864, 15204488, 15204352, 8388704,
      22544480, 12583064, 21495848, 22020336, 27787608, 13107264, 0, 0, 27263152, 17826040, 9437192, 14155936, 14155808, 24641576, 19398768, 26214688,
      12058656, 18350104, 26214544, 19922976, 22544400, 19923216, 0, 0, 11534336, 8912984, 15728704, 16777264, 0, 0, 0, 0,
      4718600, 24117264, 9437296, 11534440, 12582968, 25165912, 9961584, 26738776, 13107392, 15728744, 22020152, 14680136, 13107296, 12058632, 12058712, 17825936,
      20971656, 17301528, 16777288, 23068848, 27787504, 27263376, 0, 0, 24641568, 26738728, 26738864, 25690136, 21496072, 16253096, 23593008, 17825992,
      5767240, 4194368, 23593064, 25690264, 18874480, 13107344, 27263264, 23593240, 25690184, 25165952, 22020288, 22544472, 0, 0, 0, 0,
      19923072, 25166160, 27263312, 12058800, 22020312, 12582944, 12058784, 26214688, 19398752, 26214784, 10485784, 26214472, 26214600, 24641608, 19922952, 13107256,
      12582952, 20971696, 14680272, 21495872, 0, 0, 0, 0, 24117368, 9437288, 23593264, 17301768, 17301592, 8388736, 9437320, 13107280,
      9961616, 26214568, 25166016, 13107368, 27262976, 12058632, 18350144, 18874408, 26739032, 25166056, 25165952, 16252984, 0, 0, 0, 0,
      20447312, 18350184, 17301608, 25165952, 6291528, 7340032, 23593064, 27263272, 11010056, 27263136, 20447320, 14155896, 0, 0, 12058744, 13631552,
      27263160, 24641776, 19923040, 9961576, 524296, 27787672, 0, 0, 17301712, 16777400, 6815768, 26214512, 14155968, 20971832, 22020160, 14680152,
      26214480, 4194360, 19923072, 18874432, 0, 0, 7340144, 20971672, 13631560, 13107320, 8913016, 22544384, 27787440, 20971520, 0, 0,
      18874568, 23593264, 2621448, 9961496, 25690184, 16777216, 14155832, 24641608, 8388608, 19922960, 18350344, 20447536, 26739008, 15204360, 26738768, 26214784,
      16252976, 15204464, 17301736, 15728744, 0, 0, 0, 0, 16777448, 16253120, 16777240, 14155920, 9961488, 26214496, 15204416, 11534448,
      27263088, 15728736, 9961616, 23068712, 17301728, 18874432, 20447312, 26214656, 5242912, 10485800, 17825952, 7340104, 24117344, 27787528, 0, 0,
      24117528, 20447392, 19398832, 18350160, 18874560, 21495912, 23068888, 27263272, 19922992, 17825872, 19398696, 14680216, 23593200, 27263224, 27263272, 17301704,
      11534472, 9961600, 18350232, 19923160, 0, 0, 0, 0, 22544400, 8388720, 0, 0, 23068736, 18350240, 12058784, 18350136,
      13107312, 25690136, 16777240, 22544480, 23068760, 22544440, 17301720, 20447384, 24641712, 16252952, 11534368, 17826016, 27787512, 26214760, 0, 0,
      13631504, 12058736, 23592992, 27263048, 25165864, 7864328, 21495832, 15728704, 12058784, 11010048, 16253040, 13107392, 11010064, 18874392, 7864376, 19398744,
      21495960, 16253056, 22020344, 21495872, 0, 0, 0, 0, 19398704, 11534336, 0, 0, 8913008, 6815840, 8912968, 6815744,
      19923056, 23068712, 0, 0, 18874504, 23068824, 0, 0, 24641600, 18350096, 26738912, 23068696, 0, 0, 0, 0,
      15728720, 12058768, 20447304, 24641680, 27263016, 17825976, 25690296, 20447496, 23593032, 26738832, 14680280, 26214592, 12058808, 25690384, 19923216, 11010072,
      10485888, 6815824, 11534488, 12058688, 0, 0, 0, 0, 26738752, 26214600, 20971632, 14155864, 27263200, 25690152, 19923168, 22020392,
      22544664, 13631632, 16253160, 27263320, 21495992, 16253120, 22020376, 14680256, 27263256, 16253144, 26738856, 25690264, 0, 0, 0, 0,
      25166144, 22544392, 12058712, 15204416, 24117464, 26738816, 24117520, 9961584, 18350096, 13107232, 24117296, 8388624, 25166000, 24117440, 14155912, 27262976,
      16253120, 22544696, 26738816, 17301600, 0, 0, 0, 0, 27263240, 24641784, 12058776, 15728640, 15204496, 22020408, 8388664, 10485872,
      26214792, 19398872, 11534352, 8388632, 13631688, 23593152, 9437240, 19398720, 8388656, 17825856, 18350144, 8388736, 27787600, 14680080, 0, 0,
      17301688, 25166056, 24117472, 19398720, 14155888, 20447256, 12582920, 12058776, 14155936, 24117360, 6291552, 24641552, 20447408, 27263096, 19398888, 26214656,
      8388680, 6815808, 13107304, 27263136, 18350088, 27787512, 0, 0, 17825928, 26738728, 3670040, 2097152, 23593104, 24117456, 19398832, 9437288,
      17301608, 25690184, 9437240, 24117472, 2621456, 26214448, 20447456, 23593296, 20447376, 19923184, 24641712, 12058736, 26738808, 27787592, 0, 0,
      17301664, 19398760, 16777344, 21495912, 20447304, 27263056, 5767176, 20971520, 10485768, 24117248, 24117440, 25690176, 14680256, 11010136, 17301640, 23068768,
      25690184, 23068784, 17301640, 23593016, 0, 0, 0, 0, 16777440, 11010192, 27263136, 24117432, 7340128, 26214616, 16777272, 19398936,
      23593120, 19398856, 26214664, 18874384, 26214784, 13107256, 22544448, 14680256, 17301696, 12058792, 18874584, 17301688, 0, 0, 0, 0,
      27263080, 26738880, 20971832, 17826040, 6815808, 7864320, 11534448, 20971648, 17301656, 18874464, 13107384, 27263080, 18350152, 20971816, 21495904, 20447360,
      18350112, 17301544, 17301608, 23593040, 27787608, 11010064, 0, 0, 19923016, 10485888, 25690328, 24641784, 26738912, 24117360, 0, 0,
      7864416, 26214592, 22544480, 15204456, 26214784, 17301504, 25165912, 20971816, 26214608, 13107376, 19923064, 22020384, 24117264, 27787368, 0, 0,
      25165864, 17301536, 16253080, 18350280, 22544400, 17301544, 24641616, 18350080, 24117568, 12058696, 8913008, 24641608, 22020400, 14680208, 22020104, 26214528,
      18874496, 17301648, 24117456, 19398896, 5767176, 27787440, 0, 0, 24117504, 19398904, 11010080, 9961592, 10485912, 8912976, 15204512, 9961616,
      25165928, 24117512, 17825928, 24641568, 14155864, 18350128, 25165912, 23068712, 8913016, 14680264, 17301768, 18874568, 6291520, 27787440, 0, 0,
      24641656, 21495824, 14155864, 12582936, 13631584, 20447344, 22544584, 17301696, 0, 0, 13631592, 16253056, 25690264, 27263272, 7340104, 22020104,
      9437192, 13107272, 15728752, 27263152, 27787608, 18874392, 0, 0, 4718624, 5242904, 19398888, 11010200, 19923104, 19398736, 0, 0,
      17301616, 26214648, 12058712, 11534448, 16253008, 25165944, 11010136, 22544448, 16777224, 24641824, 24641656, 14155920, 27787568, 5242888, 0, 0,
      438835728, 433592792, 431495600, 452991568, 452991368, 429922672, 449321328, 435165656, 451943088, 447224248, 449321424, 451418600, 450370072, 447224464, 428874104, 435689864,
      426776944, 426776944, 448272808, 437787096, 454564352, 434117032, 0, 0, 447748728, 441981400, 452467160, 450894440, 437787128, 447224336, 454040208, 447224440,
      445651528, 445127224, 445651600, 449845784, 443029904, 449321424, 442505712, 447748712, 439359984, 443029960, 446700072, 452467120, 439884160, 454564392, 0, 0,
      439360040, 454040040, 438835672, 449845888, 452467088, 444078560, 443029976, 443554312, 426776944, 426776944, 445127224, 450370032, 454040216, 453515800, 439884232, 444078488,
      436738480, 436214144, 449321600, 442505672, 426776944, 426776944, 0, 0, 450369952, 451418800, 433068488, 436738456, 436738568, 435165560, 447748680, 444602920,
      433592792, 445127080, 450369976, 444078600, 450370056, 443029880, 446175840, 445127288, 440408496, 449321440, 440932752, 447748560, 426776944, 426776944, 0, 0,
      440408432, 452467088, 451942840, 439884304, 454039976, 453515760, 443554312, 445127288, 449321648, 439360032, 437262800, 436738472, 453515808, 441981432, 441981296, 435165648,
      449321424, 439360008, 448272792, 448797280, 454564552, 439884208, 0, 0, 454040096, 444602984, 436214136, 440932880, 440932752, 451418520, 446175712, 452991632,
      438835600, 445127048, 452991488, 446699920, 449321344, 446700160, 426776944, 426776944, 438311280, 435689928, 442505648, 443554208, 426776944, 426776944, 0, 0,
      431495544, 450894208, 436214240, 438311384, 439359912, 451942856, 436738528, 453515720, 439884336, 442505688, 448797096, 441457080, 439884240, 438835576, 438835656, 444602880,
      447748600, 444078472, 443554232, 449845792, 454564448, 454040320, 0, 0, 451418512, 453515672, 453515808, 452467080, 448273016, 443030040, 450369952, 444602936,
      432544184, 430971312, 450370008, 452467208, 445651424, 439884288, 454040208, 450370184, 452467128, 451942896, 448797232, 449321416, 426776944, 426776944, 0, 0,
      446700016, 451943104, 454040256, 438835744, 448797256, 439359888, 438835728, 452991632, 446175696, 452991728, 437262728, 452991416, 452991544, 451418552, 446699896, 439884200,
      439359896, 447748640, 441457216, 448272816, 426776944, 426776944, 0, 0, 450894312, 436214232, 450370208, 444078712, 444078536, 435165680, 436214264, 439884224,
      436738560, 452991512, 451942960, 439884312, 454039920, 438835576, 445127088, 445651352, 453515976, 451943000, 451942896, 443029928, 426776944, 426776944, 0, 0,
      447224256, 445127128, 444078552, 451942896, 433068472, 434116976, 450370008, 454040216, 437787000, 454040080, 447224264, 440932840, 426776944, 426776944, 438835688, 440408496,
      454040104, 451418720, 446699984, 436738520, 427301240, 454564616, 0, 0, 444078656, 443554344, 433592712, 452991456, 440932912, 447748776, 448797104, 441457096,
      452991424, 430971304, 446700016, 445651376, 426776944, 426776944, 434117088, 447748616, 440408504, 439884264, 435689960, 449321328, 454564384, 447748464, 0, 0,
      445651512, 450370208, 429398392, 436738440, 452467128, 443554160, 440932776, 451418552, 435165552, 446699904, 445127288, 447224480, 453515952, 441981304, 453515712, 452991728,
      443029920, 441981408, 444078680, 442505688, 426776944, 426776944, 0, 0, 443554392, 443030064, 443554184, 440932864, 436738432, 452991440, 441981360, 438311392,
      454040032, 442505680, 436738560, 449845656, 444078672, 445651376, 447224256, 452991600, 432019856, 437262744, 444602896, 434117048, 450894288, 454564472, 0, 0,
      450894472, 447224336, 446175776, 445127104, 445651504, 448272856, 449845832, 454040216, 446699936, 444602816, 446175640, 441457160, 450370144, 454040168, 454040216, 444078648,
      438311416, 436738544, 445127176, 446700104, 426776944, 426776944, 0, 0, 449321344, 435165664, 426776944, 426776944, 449845680, 445127184, 438835728, 445127080,
      439884256, 452467080, 443554184, 449321424, 449845704, 449321384, 444078664, 447224328, 451418656, 443029896, 438311312, 444602960, 454564456, 452991704, 0, 0,
      440408448, 438835680, 450369936, 454039992, 451942808, 434641272, 448272776, 442505648, 438835728, 437786992, 443029984, 439884336, 437787008, 445651336, 434641320, 446175688,
      448272904, 443030000, 448797288, 448272816, 426776944, 426776944, 0, 0, 446175648, 438311280, 426776944, 426776944, 435689952, 433592784, 435689912, 433592688,
      446700000, 449845656, 426776944, 426776944, 445651448, 449845768, 426776944, 426776944, 451418544, 445127040, 453515856, 449845640, 426776944, 426776944, 0, 0,
      442505664, 438835712, 447224248, 451418624, 454039960, 444602920, 452467240, 447224440, 450369976, 453515776, 441457224, 452991536, 438835752, 452467328, 446700160, 437787016,
      437262832, 433592768, 438311432, 438835632, 426776944, 426776944, 0, 0, 453515696, 452991544, 447748576, 440932808, 454040144, 452467096, 446700112, 448797336,
      449321608, 440408576, 443030104, 454040264, 448272936, 443030064, 448797320, 441457200, 454040200, 443030088, 453515800, 452467208, 426776944, 426776944, 0, 0,
      451943088, 449321336, 438835656, 441981360, 450894408, 453515760, 450894464, 436738528, 445127040, 439884176, 450894240, 435165568, 451942944, 450894384, 440932856, 454039920,
      443030064, 449321640, 453515760, 444078544, 426776944, 426776944, 0, 0, 454040184, 451418728, 438835720, 442505584, 441981440, 448797352, 435165608, 437262816,
      452991736, 446175816, 438311296, 435165576, 440408632, 450370096, 436214184, 446175664, 435165600, 444602800, 445127088, 435165680, 454564544, 441457024, 0, 0,
      444078632, 451943000, 450894416, 446175664, 440932832, 447224200, 439359864, 438835720, 440932880, 450894304, 433068496, 451418496, 447224352, 454040040, 446175832, 452991600,
      435165624, 433592752, 439884248, 454040080, 445127032, 454564456, 0, 0, 444602872, 453515672, 430446984, 428874096, 450370048, 450894400, 446175776, 436214232,
      444078552, 452467128, 436214184, 450894416, 429398400, 452991392, 447224400, 450370240, 447224320, 446700128, 451418656, 438835680, 453515752, 454564536, 0, 0,
      444078608, 446175704, 443554288, 448272856, 447224248, 454040000, 432544120, 447748464, 437262712, 450894192, 450894384, 452467120, 441457200, 437787080, 444078584, 449845712,
      452467128, 449845728, 444078584, 450369960, 426776944, 426776944, 0, 0, 443554384, 437787136, 454040080, 450894376, 434117072, 452991560, 443554216, 446175880,
      450370064, 446175800, 452991608, 445651328, 452991728, 439884200, 449321392, 441457200, 444078640, 438835736, 445651528, 444078632, 426776944, 426776944, 0, 0,
      454040024, 453515824, 447748776, 444602984, 433592752, 434641264, 438311392, 447748592, 444078600, 445651408, 439884328, 454040024, 445127096, 447748760, 448272848, 447224304,
      445127056, 444078488, 444078552, 450369984, 454564552, 437787008, 0, 0, 446699960, 437262832, 452467272, 451418728, 453515856, 450894304, 426776944, 426776944,
      434641360, 452991536, 449321424, 441981400, 452991728, 444078448, 451942856, 447748760, 452991552, 439884320, 446700008, 448797328, 450894208, 454564312, 0, 0,
      451942808, 444078480, 443030024, 445127224, 449321344, 444078488, 451418560, 445127024, 450894512, 438835640, 435689952, 451418552, 448797344, 441457152, 448797048, 452991472,
      445651440, 444078592, 450894400, 446175840, 432544120, 454564384, 0, 0, 450894448, 446175848, 437787024, 436738536, 437262856, 435689920, 441981456, 436738560,
      451942872, 450894456, 444602872, 451418512, 440932808, 445127072, 451942856, 449845656, 435689960, 441457208, 444078712, 445651512, 433068464, 454564384, 0, 0,
      451418600, 448272768, 440932808, 439359880, 440408528, 447224288, 449321528, 444078640, 426776944, 426776944, 440408536, 443030000, 452467208, 454040216, 434117048, 448797048,
      436214136, 439884216, 442505696, 454040096, 454564552, 445651336, 0, 0, 431495568, 432019848, 446175832, 437787144, 446700048, 446175680, 426776944, 426776944,
      444078560, 452991592, 438835656, 438311392, 443029952, 451942888, 437787080, 449321392, 443554168, 451418768, 451418600, 440932864, 454564512, 432019832, 0, 0};
  alignas(16) static constexpr uint32_t kTm[1536] = {
      252708552, 389024032, 325062336, 177213368, 405280296, 165680336, 79172656, 110625728, 49808120, 320868120, 278924912, 88083280, 76552248, 146802824, 176165688, 147328024,
      367005480, 42992848, 331878576, 407899000, 398989392, 212862368, 212864176, 212864176, 310383704, 78647936, 297275256, 70783288, 263719488, 57676704, 184554320, 28311984,
      179311392, 126353848, 293079648, 90705856, 69212216, 255332208, 48235120, 33556352, 404227552, 87559304, 33032976, 212864176, 212864176, 212864176, 212864176, 212864176,
      196087808, 364910016, 346035272, 325062896, 128453136, 89653800, 62915584, 316672792, 50856496, 315623880, 77595984, 106957424, 191370216, 76027480, 305664752, 286789528,
      408424856, 85463344, 212865424, 212864176, 212864176, 212864176, 212864176, 212864176, 119539400, 46663944, 282068376, 60297904, 332400360, 61344512, 189272136, 89130176,
      90179280, 322439712, 51386360, 276828288, 153620888, 343937416, 164632536, 269486136, 290461416, 376968536, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176,
      196610680, 34082680, 110105000, 351802088, 341841144, 362285048, 352322760, 241702328, 36704024, 268960496, 90178624, 191369720, 58198848, 311432248, 299893312, 242747360,
      192417808, 393221816, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 127932336, 190322288, 78646104, 50337528, 122684496, 331355976, 63963688, 113250832,
      387452968, 245893608, 147855368, 169869960, 159386000, 63440256, 386929352, 66585592, 123210288, 212866416, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176,
      56629264, 288888720, 87037360, 135792392, 101190608, 156764016, 174065920, 183501648, 258479744, 297801456, 99091944, 188748000, 372247128, 298846632, 376969552, 187697848,
      212864768, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 153094384, 409995240, 198183032, 326633040, 178260488, 47187176, 59773664, 108529400,
      95946544, 353375608, 177738808, 311956632, 83364488, 194517016, 247993512, 38277720, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176,
      395842432, 126879456, 287839544, 53479056, 95424352, 381685944, 260573856, 186125976, 387450472, 258479776, 388499184, 374870008, 312479552, 84938952, 300946168, 212862960,
      212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 366481168, 74450176, 140514480, 277349168, 385880432, 136318888, 284693200, 100666336,
      271585080, 125832096, 244320072, 190841280, 156239136, 362809504, 343414456, 212865280, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176,
      127929080, 386402744, 342884952, 59246248, 170399432, 138938952, 136319048, 58724728, 333972456, 45613720, 207624416, 130553184, 30938112, 401082928, 146276888, 212864176,
      212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 212864176, 336071384, 382206896, 295702144, 250614488, 144185104, 212863080, 386406000, 338171696,
      354944832, 155715656, 278401968, 281020208, 139989528, 109580504, 396362368, 164627440, 311953784, 97521272, 380110928, 94372376, 212861856, 212864176, 212864176, 212864176,
      82839832, 275252904, 68686608, 355468792, 338694848, 50857792, 116392624, 160435168, 99620160, 203949704, 74975504, 328210240, 346556768, 38274264, 212863080, 212864176,
      46140128, 119015792, 188224736, 160959088, 283117240, 137889336, 212865496, 212864176, 132651112, 177210776, 148901776, 370152112, 51910488, 332403744, 54528144, 90702456,
      387977112, 328204864, 296748608, 195563792, 163579464, 287310328, 300423048, 57677056, 183506792, 278921888, 69211704, 384306280, 212863792, 212864176, 212864176, 212864176,
      128453344, 383784216, 265819272, 304087792, 37230624, 262149848, 305666040, 195035872, 244324320, 97520264, 210765080, 211293448, 166729360, 415241232, 247469144, 381685384,
      250087680, 396892232, 290985600, 390075664, 73926216, 212864176, 212864176, 212864176, 96999440, 363861304, 326636296, 385876768, 59774464, 95947320, 389547048, 147326352,
      80746776, 33555928, 86513624, 91755464, 144181480, 249041664, 152573848, 333449944, 265290248, 392171560, 254805184, 68161360, 157290888, 248517168, 212864176, 212864176,
      120065920, 70780856, 68684144, 180883640, 337123256, 339743768, 290981400, 189797256, 109054160, 372773544, 322967760, 378016616, 288363672, 212867408, 181408664, 88607080,
      369105168, 357044136, 297796080, 373819808, 279451552, 401081432, 212863880, 212864176, 285737800, 106434624, 117441240, 335022664, 394265368, 320344448, 309334208, 286789776,
      279450056, 186652128, 299369592, 405804552, 195564880, 212865112, 181409680, 349701424, 102239120, 360716440, 174594136, 98569976, 185598808, 180357632, 212866416, 212864176,
      56628184, 142611928, 106431744, 265816408, 274728264, 108530576, 78123552, 154144496, 43518344, 360714920, 370672240, 91751712, 343410848, 212865424, 168825424, 39847888,
      28840032, 55576456, 361236984, 335546384, 286266904, 398987728, 212864720, 212864176, 163054408, 341839744, 330831256, 350226544, 65015816, 374342920, 154145440, 360191552,
      182977760, 375394480, 424153640, 165156176, 274205376, 212864176, 46141216, 148899904, 131601488, 82314440, 302520272, 58721344, 173540896, 30935848, 368580472, 212864176,
      385356200, 317198928, 89653976, 47190824, 241702864, 329779736, 320344880, 42472328, 100667744, 254280744, 299896880, 290458464, 35652536, 212864176, 74454480, 44567104,
      52433600, 382733480, 78121856, 306710048, 365434208, 251137720, 77071608, 212864176, 319819840, 30410816, 124782312, 103288952, 189269608, 388503200, 48763384, 281546608,
      179836248, 212862024, 292031056, 129500968, 411569888, 425202832, 339740712, 380639544, 185076168, 182980936, 378016616, 162010672, 310904648, 393740880, 307761920, 212864176,
      340266784, 371724528, 379066408, 131077200, 383260608, 391124208, 300945840, 369624216, 165154928, 212863152, 133698984, 391647120, 414718136, 244847400, 212342624, 303563824,
      373819808, 264770232, 421004232, 130549776, 304613344, 424149584, 212866408, 212864176, 82842784, 390596856, 135792392, 211814264, 178786672, 309332016, 326112112, 282592896,
      128980208, 362813488, 247991192, 193463512, 140510336, 117441432, 364382728, 257426480, 367531968, 112202560, 421529768, 29366096, 246421600, 212867136, 212864176, 212864176,
      31982184, 63964240, 201331848, 380639232, 403183600, 262148416, 81789568, 421532872, 104863176, 251660224, 365955664, 371200296, 95425816, 79172536, 272106656, 67637240,
      159384896, 153617504, 246945568, 72878000, 62392080, 212861472, 212864176, 212864176, 126878296, 59248288, 383779272, 178784152, 257427296, 54531824, 306714656, 84935640,
      167773872, 133175392, 75501928, 103809968, 243799216, 108004352, 361237256, 37225320, 93325448, 68162248, 91226968, 156239160, 201856656, 212864176, 212864176, 212864176,
      103811704, 273679864, 350750832, 179307432, 209716984, 65542144, 112722552, 375395000, 275780712, 130025792, 300422112, 44568680, 170396128, 265292960, 137365032, 188223424,
      270537640, 51380968, 98042976, 145754432, 60819288, 212864176, 212864176, 212864176, 342888096, 30412776, 273682272, 105908120, 276305792, 57153232, 277878584, 400557040,
      42996368, 359139032, 270010144, 371197664, 335025360, 354944872, 207098368, 143657288, 401610664, 84411056, 289410864, 158862120, 285215384, 212864176, 212864176, 212864176,
      331355560, 397936600, 263197184, 357046624, 255856296, 316150112, 101716720, 186649192, 118490840, 393221624, 406848016, 212864176, 297276288, 191891816, 266866304, 113251232,
      263197088, 321918168, 139987840, 343936040, 318248040, 34605288, 212865312, 212864176, 285741080, 323490824, 124261416, 110626416, 407372256, 106959368, 256902280, 45619408,
      423625592, 249038928, 73928368, 212864176, 151523328, 323487872, 308806088, 180885144, 242225536, 67637304, 92277128, 310908104, 252183920, 146278896, 212864008, 212864176,
      50337712, 355471976, 324013960, 283640416, 167252912, 32508392, 374342624, 356521536, 145229296, 256379152, 352849672, 212864176, 149949176, 96996272, 191894424, 303042696,
      101189752, 337647120, 136845160, 114299032, 367530016, 86512072, 212865584, 212864176, 122689648, 249565392, 125309704, 31462544, 350751832, 250087264, 44043392, 289933880,
      423626256, 336595392, 212866336, 212864176, 332923496, 31982280, 150476680, 283641624, 284690968, 76548504, 146802232, 264768128, 256377816, 354424488, 212862024, 212864176,
      679485496, 815800976, 751839280, 603990312, 832057240, 592457280, 505949600, 537402672, 476585064, 747645064, 705701856, 514860224, 503329192, 573579768, 602942632, 574104968,
      793782424, 469769792, 758655520, 834675944, 825766336, 639639312, 639641120, 639641120, 737160648, 505424880, 724052200, 497560232, 690496432, 484453648, 611331264, 455088928,
      606088336, 553130792, 719856592, 517482800, 495989160, 682109152, 475012064, 460333296, 831004496, 514336248, 459809920, 639641120, 639641120, 639641120, 639641120, 639641120,
      622864752, 791686960, 772812216, 751839840, 555230080, 516430744, 489692528, 743449736, 477633440, 742400824, 504372928, 533734368, 618147160, 502804424, 732441696, 713566472,
      835201800, 512240288, 639642368, 639641120, 639641120, 639641120, 639641120, 639641120, 546316344, 473440888, 708845320, 487074848, 759177304, 488121456, 616049080, 515907120,
      516956224, 749216656, 478163304, 703605232, 580397832, 770714360, 591409480, 696263080, 717238360, 803745480, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120,
      623387624, 460859624, 536881944, 778579032, 768618088, 789061992, 779099704, 668479272, 463480968, 695737440, 516955568, 618146664, 484975792, 738209192, 726670256, 669524304,
      619194752, 819998760, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 554709280, 617099232, 505423048, 477114472, 549461440, 758132920, 490740632, 540027776,
      814229912, 672670552, 574632312, 596646904, 586162944, 490217200, 813706296, 493362536, 549987232, 639643360, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120,
      483406208, 715665664, 513814304, 562569336, 527967552, 583540960, 600842864, 610278592, 685256688, 724578400, 525868888, 615524944, 799024072, 725623576, 803746496, 614474792,
      639641712, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 579871328, 836772184, 624959976, 753409984, 605037432, 473964120, 486550608, 535306344,
      522723488, 780152552, 604515752, 738733576, 510141432, 621293960, 674770456, 465054664, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120,
      822619376, 553656400, 714616488, 480256000, 522201296, 808462888, 687350800, 612902920, 814227416, 685256720, 815276128, 801646952, 739256496, 511715896, 727723112, 639639904,
      639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 793258112, 501227120, 567291424, 704126112, 812657376, 563095832, 711470144, 527443280,
      698362024, 552609040, 671097016, 617618224, 583016080, 789586448, 770191400, 639642224, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120,
      554706024, 813179688, 769661896, 486023192, 597176376, 565715896, 563095992, 485501672, 760749400, 472390664, 634401360, 557330128, 457715056, 827859872, 573053832, 639641120,
      639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 639641120, 762848328, 808983840, 722479088, 677391432, 570962048, 639640024, 813182944, 764948640,
      781721776, 582492600, 705178912, 707797152, 566766472, 536357448, 823139312, 591404384, 738730728, 524298216, 806887872, 521149320, 639638800, 639641120, 639641120, 639641120,
      509616776, 702029848, 495463552, 782245736, 765471792, 477634736, 543169568, 587212112, 526397104, 630726648, 501752448, 754987184, 773333712, 465051208, 639640024, 639641120,
      472917072, 545792736, 615001680, 587736032, 709894184, 564666280, 639642440, 639641120, 559428056, 603987720, 575678720, 796929056, 478687432, 759180688, 481305088, 517479400,
      814754056, 754981808, 723525552, 622340736, 590356408, 714087272, 727199992, 484454000, 610283736, 705698832, 495988648, 811083224, 639640736, 639641120, 639641120, 639641120,
      555230288, 810561160, 692596216, 730864736, 464007568, 688926792, 732442984, 621812816, 671101264, 524297208, 637542024, 638070392, 593506304, 842018176, 674246088, 808462328,
      676864624, 823669176, 717762544, 816852608, 500703160, 639641120, 639641120, 639641120, 523776384, 790638248, 753413240, 812653712, 486551408, 522724264, 816323992, 574103296,
      507523720, 460332872, 513290568, 518532408, 570958424, 675818608, 579350792, 760226888, 692067192, 818948504, 681582128, 494938304, 584067832, 675294112, 639641120, 639641120,
      546842864, 497557800, 495461088, 607660584, 763900200, 766520712, 717758344, 616574200, 535831104, 799550488, 749744704, 804793560, 715140616, 639644352, 608185608, 515384024,
      795882112, 783821080, 724573024, 800596752, 706228496, 827858376, 639640824, 639641120, 712514744, 533211568, 544218184, 761799608, 821042312, 747121392, 736111152, 713566720,
      706227000, 613429072, 726146536, 832581496, 622341824, 639642056, 608186624, 776478368, 529016064, 787493384, 601371080, 525346920, 612375752, 607134576, 639643360, 639641120,
      483405128, 569388872, 533208688, 692593352, 701505208, 535307520, 504900496, 580921440, 470295288, 787491864, 797449184, 518528656, 770187792, 639642368, 595602368, 466624832,
      455616976, 482353400, 788013928, 762323328, 713043848, 825764672, 639641664, 639641120, 589831352, 768616688, 757608200, 777003488, 491792760, 801119864, 580922384, 786968496,
      609754704, 802171424, 850930584, 591933120, 700982320, 639641120, 472918160, 575676848, 558378432, 509091384, 729297216, 485498288, 600317840, 457712792, 795357416, 639641120,
      812133144, 743975872, 516430920, 473967768, 668479808, 756556680, 747121824, 469249272, 527444688, 681057688, 726673824, 717235408, 462429480, 639641120, 501231424, 471344048,
      479210544, 809510424, 504898800, 733486992, 792211152, 677914664, 503848552, 639641120, 746596784, 457187760, 551559256, 530065896, 616046552, 815280144, 475540328, 708323552,
      606613192, 639638968, 718808000, 556277912, 838346832, 851979776, 766517656, 807416488, 611853112, 609757880, 804793560, 588787616, 737681592, 820517824, 734538864, 639641120,
      767043728, 798501472, 805843352, 557854144, 810037552, 817901152, 727722784, 796401160, 591931872, 639640096, 560475928, 818424064, 841495080, 671624344, 639119568, 730340768,
      800596752, 691547176, 847781176, 557326720, 731390288, 850926528, 639643352, 639641120, 509619728, 817373800, 562569336, 638591208, 605563616, 736108960, 752889056, 709369840,
      555757152, 789590432, 674768136, 620240456, 567287280, 544218376, 791159672, 684203424, 794308912, 538979504, 848306712, 456143040, 673198544, 639644080, 639641120, 639641120,
      458759128, 490741184, 628108792, 807416176, 829960544, 688925360, 508566512, 848309816, 531640120, 678437168, 792732608, 797977240, 522202760, 505949480, 698883600, 494414184,
      586161840, 580394448, 673722512, 499654944, 489169024, 639638416, 639641120, 639641120, 553655240, 486025232, 810556216, 605561096, 684204240, 481308768, 733491600, 511712584,
      594550816, 559952336, 502278872, 530586912, 670576160, 534781296, 788014200, 464002264, 520102392, 494939192, 518003912, 583016104, 628633600, 639641120, 639641120, 639641120,
      530588648, 700456808, 777527776, 606084376, 636493928, 492319088, 539499496, 802171944, 702557656, 556802736, 727199056, 471345624, 597173072, 692069904, 564141976, 615000368,
      697314584, 478157912, 524819920, 572531376, 487596232, 639641120, 639641120, 639641120, 769665040, 457189720, 700459216, 532685064, 703082736, 483930176, 704655528, 827333984,
      469773312, 785915976, 696787088, 797974608, 761802304, 781721816, 633875312, 570434232, 828387608, 511188000, 716187808, 585639064, 711992328, 639641120, 639641120, 639641120,
      758132504, 824713544, 689974128, 783823568, 682633240, 742927056, 528493664, 613426136, 545267784, 819998568, 833624960, 639641120, 724053232, 618668760, 693643248, 540028176,
      689974032, 748695112, 566764784, 770712984, 745024984, 461382232, 639642256, 639641120, 712518024, 750267768, 551038360, 537403360, 834149200, 533736312, 683679224, 472396352,
      850402536, 675815872, 500705312, 639641120, 578300272, 750264816, 735583032, 607662088, 669002480, 494414248, 519054072, 737685048, 678960864, 573055840, 639640952, 639641120,
      477114656, 782248920, 750790904, 710417360, 594029856, 459285336, 801119568, 783298480, 572006240, 683156096, 779626616, 639641120, 576726120, 523773216, 618671368, 729819640,
      527966696, 764424064, 563622104, 541075976, 794306960, 513289016, 639642528, 639641120, 549466592, 676342336, 552086648, 458239488, 777528776, 676864208, 470820336, 716710824,
      850403200, 763372336, 639643280, 639641120, 759700440, 458759224, 577253624, 710418568, 711467912, 503325448, 573579176, 691545072, 683154760, 781201432, 639638968, 639641120};
  static constexpr int kBnd[32] = {
      0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 3, 8, 7, 7, 7,
      7, 7, 7, 7, 7, 5, 5, 6, 5, 5, 5, 5, 6, 6, 6, 6};
  // chunks at whose end some lane moves its accumulator to slot 0 (bit c)
  static constexpr uint64_t kSwitchChunks = 244ull;
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

// Wide variant: 64 lanes per system, one species per lane (rk_group.hpp).
struct WNet {
  static constexpr bool kWide = true;
  // largest batches it runs, in systems per SIMD (rk_group.hpp group_rhs_wide)
  static constexpr int kMaxRkck = 16;
  static constexpr int kMaxRkc = 1;
  static constexpr int N = 53;
  static constexpr int NR = 325;
  static constexpr int kL = 64;
  static constexpr int kGroupLanes = 64;
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  static constexpr int kWavesPerEuRkc = 1;
  static constexpr int kWavesPerEuRkck = 2;
  static constexpr int S = 1;
  static constexpr int R = 6;
  static constexpr int kMSlot = 5;   // first slot that may hold a [M] reaction
  static constexpr int kOffC = 0;
  static constexpr int kOffQ = 56;
  static constexpr int kOffZero = 440;
  static constexpr int kNegOff = 448;
  static constexpr int kOffRed = 442;
  static constexpr int kLdsPerSystem = 888;
  static constexpr int kTermLen = 44;
  using Params = const double*;
  static constexpr int kSp[64] = {
      0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15,
      16, 17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31,
      32, 33, 34, 35, 36, 37, 38, 39, 40, 41, 42, 43, 44, 45, 46, 47,
      48, 49, 50, 51, 52, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1};
  static constexpr int16_t kRxOf[384] = {
      0, 45, 36, 249, 2, -1, 281, 61, 47, 105, 108, 176, -1, 292, 273, 175,
      50, 55, 213, 252, 110, 208, 269, 74, 12, 304, 320, 21, 46, 247, 49, 199,
      -1, 149, 313, 77, 63, 11, 133, 127, 238, 40, 230, 189, 88, 90, 6, 226,
      125, 299, 225, 311, 58, 190, 91, 275, 312, 13, 71, 228, 75, 150, -1, 70,
      17, 246, 62, 72, 204, 126, 220, 300, 86, 195, 76, 257, 119, 43, 26, 153,
      7, 73, 219, 59, 234, 78, 324, 60, 81, 53, 221, 187, 242, 206, 157, 229,
      -1, 3, 197, 279, -1, -1, 291, 237, 240, 163, 203, 284, 117, 307, 140, 183,
      294, 207, 303, 174, 48, 296, 10, 270, 145, 286, 1, 310, 317, 250, 223, 15,
      99, 164, 209, 262, 137, 182, 302, 301, 24, 259, 265, 14, 32, 166, -1, 97,
      160, 314, 278, 171, 139, 318, 185, -1, 274, 51, 293, 239, 202, 9, 158, 169,
      170, 214, 79, 191, 85, 297, 64, 115, 194, 100, 179, 130, 198, 298, 192, 180,
      222, 83, 248, 93, 306, 258, 156, 118, 34, 224, 309, 289, 218, 31, 315, 22,
      116, 69, 285, 241, 267, 210, 216, 316, 28, 244, 56, 264, 193, 178, 196, 277,
      121, 147, 37, 38, 42, 111, 136, 124, 33, 101, 323, 200, 154, 263, 27, 280,
      134, 57, 290, 143, 161, 141, 52, 95, 114, 256, 260, 186, 319, 87, 144, 54,
      266, 254, 20, 168, 96, 283, 233, 201, -1, 184, 82, 89, 305, -1, 129, 308,
      181, 107, 205, 94, 188, 103, 131, 102, 173, 251, 4, 253, 5, 109, 112, 16,
      29, 151, 23, 165, 227, 232, 35, 30, 146, 19, 66, 113, 138, 152, 261, 217,
      128, 135, 84, 41, 212, 120, 243, 148, 255, 67, 236, 268, 177, 272, 39, 155,
      65, 271, 172, 44, 18, 106, 68, 98, 132, 321, 287, 167, 159, 211, -1, 282,
      -1, -1, -1, -1, -1, -1, 231, -1, 80, -1, -1, -1, -1, -1, 162, -1,
      -1, -1, -1, 215, -1, -1, -1, -1, -1, 235, -1, -1, -1, 104, 25, -1,
      -1, -1, 123, 322, -1, 295, -1, -1, -1, -1, -1, 8, -1, 142, 245, -1,
      -1, -1, 92, -1, -1, -1, -1, 288, -1, -1, -1, -1, -1, 276, -1, 122};
  // LDS byte offsets within the system's area: each lane's rate operands
  // (R x 4), and the signed rates of its species in reaction order
  alignas(16) static constexpr uint16_t kOp[1536] = {
      128, 384, 56, 248, 112, 112, 152, 320, 32, 216, 96, 320, 120, 184, 64, 208,
      176, 296, 104, 144, 0, 0, 0, 0, 24, 328, 64, 240, 32, 184, 24, 280,
      64, 376, 16, 280, 144, 152, 168, 400, 128, 256, 104, 328, 0, 0, 0, 0,
      224, 312, 336, 360, 32, 360, 72, 416, 80, 376, 0, 280, 56, 256, 280, 296,
      256, 368, 248, 296, 0, 0, 0, 0, 88, 264, 128, 128, 224, 264, 64, 288,
      168, 360, 288, 312, 144, 312, 240, 304, 8, 144, 72, 200, 0, 0, 0, 0,
      72, 360, 152, 264, 88, 200, 40, 264, 88, 184, 64, 232, 208, 400, 176, 200,
      72, 304, 128, 160, 0, 0, 0, 0, 0, 0, 0, 0, 16, 168, 24, 288,
      104, 264, 80, 360, 96, 328, 128, 312, 192, 224, 88, 168, 0, 0, 0, 0,
      152, 160, 80, 136, 32, 216, 40, 376, 280, 344, 144, 208, 96, 120, 192, 400,
      88, 352, 56, 344, 248, 424, 360, 400, 48, 360, 320, 376, 120, 376, 144, 216,
      200, 400, 72, 376, 120, 304, 288, 336, 216, 320, 184, 272, 0, 0, 0, 0,
      48, 368, 16, 128, 200, 280, 128, 360, 192, 264, 168, 184, 104, 184, 272, 352,
      96, 160, 56, 152, 344, 424, 64, 200, 32, 392, 112, 264, 8, 336, 128, 400,
      120, 136, 200, 224, 184, 200, 104, 416, 152, 360, 8, 248, 0, 0, 0, 0,
      8, 160, 0, 368, 176, 376, 24, 248, 96, 112, 216, 400, 184, 184, 272, 392,
      40, 296, 152, 224, 0, 0, 0, 0, 128, 408, 96, 264, 136, 288, 152, 352,
      104, 104, 56, 280, 176, 416, 248, 272, 152, 280, 216, 304, 0, 0, 0, 0,
      0, 0, 0, 0, 8, 256, 288, 376, 104, 360, 296, 416, 136, 176, 128, 152,
      8, 304, 56, 200, 0, 0, 0, 0, 176, 384, 192, 368, 160, 232, 144, 152,
      72, 392, 112, 352, 88, 384, 40, 352, 48, 360, 200, 272, 0, 0, 0, 0,
      104, 200, 160, 416, 0, 344, 104, 128, 0, 0, 0, 0, 8, 168, 160, 416,
      96, 304, 104, 152, 240, 424, 400, 416, 192, 216, 312, 320, 128, 304, 336, 384,
      216, 224, 192, 400, 8, 88, 0, 320, 56, 336, 72, 224, 0, 0, 0, 0,
      128, 304, 64, 288, 112, 320, 88, 216, 160, 360, 200, 296, 184, 264, 232, 384,
      72, 280, 296, 320, 0, 0, 0, 0, 48, 248, 112, 232, 32, 168, 120, 152,
      16, 176, 24, 128, 24, 104, 112, 400, 72, 392, 128, 384, 0, 0, 0, 0,
      200, 208, 192, 360, 104, 416, 192, 408, 216, 352, 296, 416, 160, 184, 288, 400,
      112, 288, 144, 200, 0, 0, 0, 0, 80, 240, 144, 184, 176, 312, 120, 416,
      160, 216, 112, 368, 64, 280, 40, 288, 96, 208, 112, 312, 96, 368, 264, 424,
      72, 384, 160, 200, 216, 264, 152, 312, 192, 384, 168, 200, 104, 264, 128, 384,
      112, 216, 24, 312, 0, 0, 0, 0, 96, 296, 384, 400, 88, 312, 120, 216,
      200, 344, 192, 264, 104, 384, 264, 368, 216, 336, 32, 192, 0, 0, 0, 0,
      152, 184, 0, 240, 224, 416, 40, 392, 24, 56, 0, 32, 336, 416, 176, 184,
      32, 248, 96, 344, 0, 0, 0, 0, 136, 320, 24, 264, 136, 264, 56, 360,
      0, 0, 0, 0, 104, 264, 72, 392, 208, 264, 184, 256, 0, 0, 0, 0,
      80, 312, 256, 400, 80, 400, 56, 64, 320, 344, 176, 192, 72, 312, 80, 416,
      104, 248, 152, 256, 0, 0, 0, 0, 272, 304, 24, 168, 136, 264, 96, 352,
      320, 368, 72, 184, 144, 152, 40, 352, 64, 240, 48, 256, 8, 280, 248, 424,
      88, 216, 24, 192, 152, 152, 8, 128, 88, 216, 48, 280, 16, 40, 48, 400,
      88, 184, 144, 272, 0, 0, 0, 0, 88, 96, 40, 152, 72, 112, 8, 336,
      32, 176, 224, 272, 56, 120, 88, 296, 8, 72, 16, 368, 0, 0, 0, 0,
      216, 392, 248, 376, 80, 248, 120, 384, 176, 408, 24, 392, 56, 192, 88, 384,
      40, 384, 8, 120, 0, 0, 0, 0, 80, 408, 384, 400, 152, 264, 96, 288,
      128, 192, 88, 248, 192, 200, 104, 240, 224, 408, 24, 352, 8, 8, 408, 424,
      128, 288, 144, 264, 64, 72, 224, 400, 272, 368, 112, 152, 24, 256, 96, 344,
      96, 200, 8, 184, 16, 200, 184, 424, 112, 304, 40, 352, 192, 336, 88, 344,
      264, 328, 168, 248, 72, 136, 0, 104, 104, 392, 248, 368, 0, 0, 0, 0,
      0, 0, 0, 0, 0, 0, 0, 0, 72, 312, 144, 376, 96, 344, 104, 232,
      96, 96, 16, 376, 0, 0, 0, 0, 32, 80, 40, 160, 136, 272, 40, 408,
      192, 288, 104, 328, 88, 184, 112, 176, 72, 128, 64, 104, 0, 0, 0, 0,
      112, 296, 288, 400, 64, 352, 160, 280, 384, 400, 56, 200, 288, 416, 280, 360,
      16, 280, 32, 200, 304, 424, 8, 80, 56, 128, 112, 160, 144, 232, 312, 336,
      48, 304, 80, 272, 168, 408, 152, 392, 128, 160, 80, 104, 176, 424, 0, 320,
      0, 208, 32, 392, 0, 0, 0, 0, 192, 368, 64, 392, 40, 416, 184, 272,
      112, 176, 128, 320, 0, 0, 0, 0, 64, 280, 128, 128, 0, 0, 0, 0,
      184, 416, 240, 376, 240, 360, 248, 416, 112, 200, 24, 392, 64, 96, 176, 424,
      264, 320, 104, 232, 136, 168, 160, 312, 8, 144, 160, 216, 160, 184, 0, 168,
      152, 256, 264, 280, 0, 0, 0, 0, 232, 296, 152, 168, 48, 128, 64, 272,
      304, 360, 264, 264, 176, 296, 80, 280, 208, 224, 64, 328, 0, 0, 0, 0,
      320, 408, 8, 232, 96, 344, 120, 376, 224, 408, 112, 368, 224, 304, 296, 336,
      64, 344, 192, 224, 0, 0, 0, 0, 112, 264, 248, 400, 120, 136, 0, 344,
      56, 144, 224, 368, 160, 184, 56, 280, 16, 344, 112, 128, 0, 0, 0, 0,
      56, 216, 72, 376, 384, 400, 0, 264, 8, 192, 152, 184, 232, 248, 344, 416,
      112, 240, 176, 416, 0, 0, 0, 0, 160, 304, 80, 296, 64, 232, 112, 176,
      56, 328, 104, 168, 176, 376, 112, 184, 144, 400, 32, 304, 144, 424, 56, 112,
      56, 144, 64, 296, 160, 272, 72, 112, 16, 344, 40, 264, 64, 408, 200, 400,
      216, 288, 200, 280, 0, 0, 0, 0, 16, 344, 272, 304, 184, 304, 64, 392,
      0, 176, 88, 136, 72, 208, 120, 200, 152, 328, 128, 248, 344, 424, 16, 168,
      72, 256, 176, 352, 304, 336, 144, 224, 48, 296, 0, 176, 344, 408, 232, 384,
      112, 136, 96, 104, 120, 408, 328, 424, 112, 144, 104, 176, 0, 232, 96, 128,
      184, 392, 264, 312, 392, 400, 216, 296, 120, 376, 16, 328, 0, 0, 0, 0,
      280, 336, 192, 224, 264, 264, 200, 288, 0, 128, 16, 304, 184, 192, 120, 416,
      16, 152, 96, 400, 0, 0, 0, 0, 272, 344, 88, 240, 32, 280, 40, 264,
      72, 96, 0, 112, 96, 344, 152, 192, 136, 144, 80, 200, 0, 0, 0, 0,
      160, 264, 104, 296, 64, 152, 16, 144, 40, 384, 32, 264, 296, 416, 200, 264,
      224, 256, 144, 168, 344, 424, 24, 288, 200, 288, 304, 360, 112, 248, 192, 200,
      288, 416, 264, 312, 312, 320, 248, 272, 216, 368, 128, 408, 0, 0, 0, 0,
      0, 416, 8, 184, 24, 400, 0, 48, 8, 32, 24, 136, 280, 416, 216, 248,
      112, 136, 72, 376, 0, 0, 0, 0, 72, 88, 64, 64, 232, 264, 104, 240,
      88, 168, 64, 344, 320, 384, 8, 344, 184, 328, 192, 248, 0, 0, 0, 0,
      176, 408, 136, 232, 192, 248, 312, 344, 112, 416, 96, 240, 160, 416, 184, 368,
      56, 416, 128, 408, 0, 0, 0, 0, 232, 296, 256, 400, 72, 360, 144, 408,
      160, 184, 104, 104, 88, 384, 296, 320, 24, 256, 144, 216, 8, 88, 176, 424,
      232, 256, 192, 248, 208, 368, 240, 296, 64, 104, 0, 120, 0, 0, 0, 0,
      16, 208, 112, 184, 0, 0, 0, 0, 264, 416, 248, 376, 136, 216, 0, 416,
      72, 392, 0, 256, 288, 288, 168, 352, 144, 360, 208, 368, 0, 0, 0, 0,
      320, 384, 72, 312, 104, 208, 128, 248, 280, 368, 160, 312, 136, 272, 32, 376,
      152, 392, 296, 416, 0, 0, 0, 0, 112, 152, 88, 408, 248, 336, 64, 328,
      216, 288, 184, 264, 264, 400, 16, 288, 64, 336, 88, 224, 0, 0, 0, 0,
      104, 360, 152, 392, 128, 240, 248, 320, 8, 40, 24, 152, 40, 192, 176, 320,
      24, 160, 72, 400, 0, 0, 0, 0, 64, 208, 112, 344, 80, 312, 104, 280,
      40, 328, 240, 336, 0, 0, 0, 0, 152, 176, 64, 184, 16, 368, 104, 424,
      0, 0, 0, 0, 240, 296, 264, 280, 120, 368, 104, 144, 152, 248, 200, 280,
      0, 0, 0, 0, 0, 0, 0, 0, 32, 72, 24, 80, 224, 368, 64, 296,
      32, 376, 40, 408, 296, 416, 168, 408, 264, 280, 304, 312, 336, 424, 16, 224};
  alignas(16) static constexpr uint16_t kTm[2816] = {
      4656, 1920, 1376, 2288, 4448, 4320, 1864, 528, 1288, 4920, 1648, 1840, 1296, 1488, 5440, 1928,
      624, 2104, 2232, 1416, 5416, 3288, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6176, 864, 5360, 6104,
      6824, 6824, 4112, 6296, 4640, 3280, 2720, 5392, 1176, 4616, 5680, 5536, 1168, 6792, 768, 2568,
      2736, 5688, 2408, 7032, 5472, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6832, 512, 6464, 6408, 6352, 2456, 4392, 2712,
      3512, 4584, 2752, 6528, 3368, 2872, 1480, 5408, 1856, 7080, 1360, 5192, 5776, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 5808, 4040, 4960, 952, 632, 1040, 3408, 6520, 2792, 1000, 5704, 2728,
      6560, 5232, 1696, 1952, 2656, 968, 648, 1888, 1608, 656, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      5560, 6256, 4560, 736, 4536, 4680, 2448, 2768, 5056, 4104, 4296, 1648, 4936, 4592, 2664, 5272,
      4552, 1872, 2840, 5472, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 1224, 6160, 664, 1976,
      5544, 2136, 2184, 6304, 712, 5856, 2088, 1824, 696, 992, 1352, 5536, 1008, 5456, 6048, 5776,
      1136, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 2696, 4096, 1376, 4168, 4088, 6184, 5336, 5424,
      4856, 1680, 2192, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 448, 2592, 3352, 1560, 6200, 1144, 6512, 4312, 1744, 1152, 4384, 5384,
      5400, 2544, 5792, 2560, 5232, 5784, 4368, 2312, 5584, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4328, 1464, 6280, 5504, 5720, 456, 576, 984, 3072, 1152, 1760, 800, 1984, 2760, 1504, 2808,
      4520, 4784, 5064, 6552, 872, 872, 4816, 2984, 1272, 6400, 1896, 4888, 6888, 4944, 1320, 1432,
      5920, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4064, 4400, 2616, 2912,
      6208, 5760, 1672, 976, 4536, 912, 5448, 5928, 2520, 4192, 6296, 1312, 2168, 6344, 6216, 4784,
      2976, 5160, 5312, 4760, 6112, 4456, 5512, 784, 4984, 5816, 1528, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4224, 2176, 2776, 952, 4736, 2296, 3280, 4296,
      1512, 792, 1752, 5072, 4768, 4264, 5032, 4184, 2888, 496, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 1088, 1704, 4248, 5832, 6288, 4712, 2536, 6128, 5088, 2208, 2968, 5672,
      4456, 2200, 6008, 4576, 920, 1208, 4056, 5480, 5688, 7032, 5264, 1832, 840, 4240, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4248, 2224, 2672, 2864, 1160, 2880, 5448, 1472, 6192, 6336, 6336, 5824, 1904, 6232, 6144, 536,
      1336, 1192, 4200, 5608, 6744, 5616, 4864, 5960, 6320, 5136, 6888, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 5008, 5144, 5144, 1072,
      5632, 5152, 5504, 2864, 2776, 5728, 4512, 2504, 5736, 2608, 1912, 1912, 5752, 1816, 752, 2240,
      2760, 6272, 5704, 2496, 5096, 1736, 6328, 4688, 848, 824, 2056, 1448, 2216, 4144, 3496, 2232,
      1384, 1968, 3520, 3520, 3520, 3520, 3520, 3520, 4672, 3352, 4544, 4544, 6496, 6224, 6448, 4360,
      584, 2248, 2824, 728, 1864, 520, 1312, 6376, 2944, 2120, 936, 5488, 1712, 2648, 1576, 1624,
      4952, 2328, 4760, 1792, 4280, 6368, 4408, 6240, 4504, 6416, 5136, 1304, 4304, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 1920, 1112, 1096, 1128, 2344, 5568, 2720, 6456, 4872, 5784, 5616, 1280,
      1184, 6960, 5128, 2368, 4600, 5552, 5624, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4032, 1424, 5288, 744, 744, 1072, 6360, 2144, 2904, 512, 4272, 4160, 2824, 2928, 4312, 1024,
      6088, 6344, 2632, 4664, 4120, 1336, 2528, 2080, 1032, 2024, 2784, 1168, 5440, 4856, 472, 472,
      2856, 1608, 5024, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4808, 6496, 6448, 4744,
      4728, 4216, 6032, 880, 4872, 5664, 4632, 5128, 6472, 5816, 496, 5000, 4848, 1832, 1888, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6936, 2640, 1064, 688, 5360, 2704, 5576, 4384,
      6104, 2936, 5384, 5768, 1328, 1728, 2896, 2496, 4408, 5592, 600, 6424, 1400, 6472, 4824, 1016,
      1520, 1360, 1968, 6536, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 480, 2576, 960, 664, 1064, 6464, 5576, 1096, 928, 5768, 2608, 760,
      6064, 2264, 2688, 1712, 2560, 1808, 2080, 4776, 6568, 1952, 4752, 4752, 4504, 1120, 6384, 6152,
      6168, 2376, 1048, 4208, 6440, 4080, 6544, 4944, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      5712, 6360, 4648, 5872, 1776, 728, 4112, 608, 4896, 5496, 712, 6560, 5184, 5208, 6144, 2528,
      4376, 2096, 1232, 4432, 6000, 5896, 560, 4080, 1264, 1936, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 1536, 2288, 1992, 4680,
      2536, 4584, 760, 1816, 1632, 3368, 5848, 1720, 2896, 2440, 5680, 5480, 5080, 4848, 648, 2488,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 816, 2248, 4696, 4624, 4464, 5880, 2160, 6080,
      5912, 1840, 5664, 5280, 6568, 6368, 824, 2832, 5272, 5656, 2016, 1664, 1304, 3448, 4136, 3304,
      5416, 2464, 5192, 6872, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 1536, 3248, 5632, 2680, 5712, 1672, 5872, 5648, 5648, 5832, 864, 6288,
      2552, 6504, 5568, 5496, 5696, 2944, 2160, 5088, 2272, 1808, 5432, 2328, 2984, 2416, 5640, 4552,
      600, 5896, 2736, 5952, 4208, 1944, 5352, 4904, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      5288, 4976, 5120, 5344, 1592, 6120, 2920, 832, 5216, 5792, 1368, 4152, 5392, 592, 5320, 2032,
      1104, 4792, 2664, 2376, 2816, 5800, 5952, 1664, 552, 6048, 896, 1640, 656, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 2592, 2384, 2640, 6832,
      1744, 3072, 2768, 4608, 2344, 2520, 2600, 608, 6376, 2480, 1632, 1600, 1368, 2848, 4576, 4176,
      5640, 1544, 6320, 5800, 2016, 2888, 4144, 1344, 5112, 4440, 5224, 2336, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 5008, 6264, 4320, 5928, 1984, 6528, 4992, 6392,
      4520, 6232, 4176, 5600, 1520, 2952, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 1088, 6488, 4256, 2360, 1776, 1128, 2400, 5176, 2936, 5056, 6136, 5208,
      4152, 6432, 4592, 6240, 4368, 6248, 4704, 2584, 1552, 5200, 5000, 5528, 5264, 1016, 4240, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      2576, 5048, 2616, 4048, 4568, 5176, 1800, 6120, 5888, 3512, 832, 1328, 6392, 6312, 1200, 2968,
      6480, 5376, 1688, 2816, 1544, 4720, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4648, 584, 880, 2112,
      4344, 752, 2240, 1504, 2352, 4920, 768, 5904, 4472, 4824, 4888, 4968, 4480, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6280, 1960, 456, 5864, 1408, 1904, 6704, 5040,
      6416, 2008, 4184, 2216, 624, 1384, 1768, 840, 5024, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 448, 1424, 1704, 4976, 904, 6256, 776, 672, 4168, 1040, 2400, 2920,
      6064, 2280, 6272, 2392, 1720, 4952, 2512, 2744, 6640, 3208, 4768, 2568, 5904, 2072, 2856, 5016,
      896, 1440, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4400, 640, 2696, 5808, 2680, 6520, 6088, 4640, 2688, 6480, 6096, 1928, 6384, 888, 5584, 4480,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 480, 4488, 2384, 5120,
      6264, 4360, 5728, 688, 4744, 4728, 4568, 632, 6040, 1880, 520, 2152, 1784, 1784, 5696, 5752,
      4336, 5304, 536, 1848, 5096, 1824, 1296, 992, 4776, 1352, 3160, 1456, 4432, 4704, 2800, 1872,
      4056, 6584, 1944, 4928, 4928, 4968, 1640, 3520, 4808, 2048, 2064, 2704, 6032, 808, 2552, 2600,
      4896, 5296, 2272, 2392, 1752, 1272, 1688, 2072, 4424, 4232, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 4328, 1560, 6208, 5720, 6352, 4608, 2296, 5984, 4416, 2480, 1480, 2848,
      1232, 4936, 1488, 1456, 6792, 2800, 968, 1448, 6168, 2312, 6584, 2000, 2256, 1680, 5104, 5520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      6224, 2128, 2136, 4272, 576, 984, 2456, 3408, 5464, 1056, 1000, 6432, 6024, 6024, 1192, 5320,
      4632, 1496, 5528, 5840, 1344, 4440, 720, 2040, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6160, 1464, 5968, 2624,
      1568, 2360, 800, 5880, 2304, 4344, 1408, 1600, 6080, 792, 5424, 2200, 2424, 2512, 4200, 5040,
      848, 4472, 1616, 2000, 2960, 6072, 4304, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6176, 4160, 808, 6192, 5888, 5368, 6864, 4912,
      4664, 6112, 4376, 5336, 4280, 1856, 2008, 2584, 2840, 3000, 4232, 4904, 856, 5624, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 1392, 4224, 5760, 4048, 4696, 912, 4712, 1880, 2648, 5976, 5312, 568,
      1848, 2024, 2656, 1120, 5592, 5032, 1496, 1240, 3000, 1264, 1936, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4672, 960, 2624, 5256, 504, 4496, 4216, 1472, 6136, 4336, 5976, 568, 2424, 2784, 4352, 5248,
      2104, 5992, 2464, 1440, 3288, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 5544, 4040, 6504, 2504,
      5400, 2808, 2872, 5304, 5608, 1736, 3376, 6440, 1432, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6200, 1960, 464, 2304, 7096, 4416, 5744, 4912,
      1080, 6552, 1176, 4616, 4792, 6248, 1240, 5016, 2040, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 1392, 4656, 2224, 2672, 6408, 6656, 4392, 6992, 2544, 5824, 6952, 5936,
      936, 1288, 5408, 1208, 4864, 5960, 6400, 1896, 2320, 5248, 2408, 4424, 5104, 5224, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      816, 2048, 1160, 2184, 6128, 2728, 1576, 2088, 2440, 4816, 696, 1048, 5200, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4064, 5152, 464, 1144,
      4088, 4560, 4512, 1024, 6184, 5368, 5864, 5184, 1512, 592, 3056, 6152, 5080, 4984, 2256, 856,
      6536, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 5048, 6488, 4096, 5256, 5344, 1800, 528, 2152,
      2712, 4992, 5296, 1624, 1792, 6096, 6744, 2744, 2416, 7080, 552, 5520, 5552, 2952, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 904, 2912, 5560, 672, 504, 4624, 2448, 1056, 2752, 6456, 5064, 1728,
      5912, 5072, 1008, 784, 1280, 1768, 4600, 1528, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4032, 2144, 4496, 5328, 4192, 5736, 2112, 6304, 5216, 2352, 2632, 1080, 2208, 5672, 6008, 4880,
      616, 1184, 680, 5456, 5992, 4136, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4256, 5944, 2064, 736,
      928, 1760, 4104, 2792, 2168, 2264, 6216, 5160, 5432, 1696, 6328, 5512, 6544, 1320, 1136, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 640, 2128, 776, 4960, 5944, 2880, 1992, 5328,
      4736, 6040, 1592, 2120, 1200, 2976, 3120, 1032, 4880, 616, 2032, 3056, 680, 1552, 5600, 6424,
      888, 5112, 720, 2336, 2192, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 1224, 1976, 2904, 2928, 4464, 3240, 5848, 5936, 6312, 4120, 5376, 5280,
      1104, 920, 4352, 6960, 4264, 1400, 2488, 5920, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4488, 5968, 1568, 2176, 4448, 1112, 976, 6512, 5464, 5984, 5744, 2280, 5488, 5856, 3120, 2096,
      4688, 6000, 2832, 2056, 2320, 5656, 2368, 560, 1616, 1416, 2960, 5840, 5352, 6072, 4720, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520};
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

}  // namespace gen_n53r325_7a51609a

template <>
struct FastVariant<gen_n53r325_7a51609a::Net> {
  using type = gen_n53r325_7a51609a::GNet;
};

}  // namespace rkmi
