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
  // three waves per SIMD: the evaluation loop fits 168 registers (the power
  // method and the set-up of a system run out of line)
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
  static constexpr int kTermBits = 10;
  static constexpr int kTermsPerWord = 3;
  static constexpr int kTermWords = 16;
  static constexpr int kTermLen = 48;
  static constexpr int kChunk = 4;
  using Params = const double*;
  static constexpr int kSp[64] = {
      -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, 6, 50, 18, 22, 35,
      12, 27, 37, 11, 20, 49, 17, 36, 51, 47, 21, 4, 38, 46, 48, 2,
      33, 13, 14, 19, 23, 16, 8, 25, 9, 52, 31, 24, 44, 41, 26, 32,
      42, 30, 29, 34, 10, 43, 1, 15, 39, 0, 3, 28, 45, 40, 7, 5};
  static constexpr int16_t kRxOf[352] = {
      0, 1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15, 16,
      17, 18, 19, 20, 21, 22, 23, 24, 26, 27, 28, 29, 30, 31, 32, 33,
      34, 35, 36, 37, 38, 39, 40, 41, 42, 43, 44, 45, 46, 47, 48, 49,
      50, 51, 52, 53, 54, 55, 56, 57, 58, 59, 60, 61, 62, 63, 64, 65,
      66, 67, 68, 69, 70, 71, 72, 73, 74, 75, 76, 77, 78, 79, 81, 82,
      83, 84, 85, 86, 87, 88, 89, 90, 91, 93, 94, 95, 96, 97, 98, 99,
      100, 101, 102, 103, 105, 106, 107, 108, 109, 110, 111, 112, 113, 114, 115, 116,
      117, 118, 119, 120, 121, 124, 125, 126, 127, 128, 129, 130, 131, 132, 133, 134,
      135, 136, 137, 138, 139, 140, 141, 143, 144, 145, 146, 147, 148, 149, 150, 151,
      152, 153, 154, 155, 156, 157, 158, 159, 160, 161, 163, 164, 165, 166, 167, 168,
      169, 170, 171, 172, 173, 174, 175, 176, 177, 178, 179, 180, 181, 182, 183, 184,
      185, 186, 187, 188, 189, 190, 191, 192, 193, 194, 195, 196, 197, 198, 199, 200,
      201, 202, 203, 204, 205, 206, 207, 208, 209, 210, 211, 212, 213, 214, 216, 217,
      218, 219, 220, 221, 222, 223, 224, 225, 226, 227, 228, 229, 230, 232, 233, 234,
      236, 237, 238, 239, 240, 241, 242, 243, 244, 246, 247, 248, 249, 250, 251, 252,
      253, 254, 255, 256, 257, 258, 259, 260, 261, 262, 263, 264, 265, 266, 267, 268,
      269, 270, 271, 272, 273, 274, 275, 277, 278, 279, 280, 281, 282, 283, 284, 285,
      286, 287, 289, 290, 291, 292, 293, 294, 296, 297, 298, 299, 300, 301, 302, 303,
      304, 305, 306, 307, 308, 309, 310, 311, 312, 313, 314, 315, 316, 317, 318, 319,
      320, 321, 323, 324, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1,
      8, 25, 80, 92, 104, 122, 123, 142, 162, 215, 231, 235, 245, 276, 288, 295,
      322, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1};
  // lane r's operand codes and packed term codes, each lane's contiguous and
  // 16-byte aligned (read as whole vectors at every evaluation)
  static constexpr int kRxWords = 12;
  static constexpr int kTcWords = 16;
  alignas(16) static constexpr uint32_t kRx[384] = {
      520564752, 251661576, 571610891, 773591559, 218632201, 521480481, 673525771, 873864718, 503322387, 352527906, 235353362, 0, 521148941, 722214660, 269363970, 738530066,
      387331114, 789718793, 822293270, 570953734, 856829193, 672536581, 890706178, 0, 554904841, 757737244, 856699911, 571942939, 487069451, 772676372, 553660976, 486617896,
      420090385, 285410305, 419968299, 0, 855974417, 841226004, 840241938, 353049624, 251736069, 353509404, 553982219, 572265988, 521152787, 822617623, 604189995, 0,
      471016709, 604316424, 167971076, 554578180, 420818968, 319230988, 622800416, 789523212, 873732365, 857027621, 892535041, 0, 419898881, 218894606, 654913576, 521677079,
      470952486, 421011214, 604774675, 639510290, 404106024, 655633955, 469906730, 0, 739647497, 840900878, 604512540, 688726032, 874458398, 673651480, 553984772, 806297354,
      840967453, 688400927, 167851302, 0, 453715982, 218764304, 319755524, 771757057, 823341845, 554447632, 842016012, 589373459, 671091457, 757474329, 352466219, 0,
      520820752, 806363405, 553854993, 572075270, 807220011, 588850203, 587214602, 873273623, 874851355, 521674781, 875705630, 0, 723984152, 319954196, 823340301, 420753417,
      622734874, 738537483, 655370508, 587405060, 707206418, 841229582, 891366924, 0, 269493000, 856698395, 520302358, 773926925, 538124045, 387127297, 386405907, 842019594,
      218108169, 268637698, 841823519, 0, 840967946, 503851267, 336465927, 319628812, 839781635, 656486679, 672142862, 553922565, 285873171, 302853647, 891233025, 0,
      790574113, 790573339, 453977867, 771885313, 688397338, 302851350, 756554265, 269492491, 656810785, 707012111, 891892495, 0, 587664653, 268578310, 419902000, 707077660,
      335874564, 755638541, 688727064, 588064522, 721498152, 673127952, 890056194, 0, 621293084, 100676099, 134689290, 555822374, 722344456, 269229312, 840437516, 520170771,
      370023688, 555232025, 890637057, 0, 470362631, 554837008, 788800017, 436737807, 806367497, 739583012, 773796109, 387063306, 623058951, 840512264, 890637320, 0,
      672337422, 604513808, 234884105, 235479572, 738407196, 67110659, 318964993, 639312659, 872422161, 402856715, 671102230, 0, 789123342, 386477608, 419701506, 218961684,
      808068624, 386805526, 857224205, 403909388, 874852627, 773467410, 0, 0, 537271816, 352327444, 822619672, 790896641, 806033415, 704712201, 788863748, 471345928,
      555164699, 839255298, 0, 0, 555299877, 738992401, 756032281, 822286606, 688008975, 336602633, 268505875, 587667220, 757281828, 822424604, 0, 0,
      319097867, 622539313, 420420105, 807215383, 504116238, 621422100, 637669376, 739451921, 655627537, 0, 0, 0, 855977732, 487464710, 621285895, 822681869,
      840698120, 134744841, 589374750, 721949963, 773337110, 0, 0, 0, 420619278, 824317719, 604123681, 471345699, 319696418, 571090438, 536883465, 471404815,
      587602699, 0, 0, 0, 387260696, 370022155, 639773442, 604181762, 839455747, 369108230, 621617428, 875241245, 605626657, 0, 0, 0,
      269298432, 385954816, 487666454, 353576221, 622406932, 319821329, 369955342, 385947916, 504176925, 0, 0, 0, 722214915, 873408278, 656487460, 788663308,
      571945989, 772682524, 654514958, 656682261, 790508567, 0, 0, 0, 740431629, 755441937, 420024833, 588848915, 721424655, 839920129, 856363790, 504174872,
      285939200, 0, 0, 0, 673522441, 791162118, 587867414, 353184007, 587345672, 873731329, 722151960, 572470294, 504048418, 0, 0, 0,
      538386714, 873016580, 521876515, 721890315, 655235596, 588524552, 789125895, 840633868, 454176527, 0, 0, 0, 706619653, 822352384, 840440859, 386800130,
      739127561, 553986818, 402926107, 873404439, 789131801, 0, 0, 0, 874851597, 454300161, 454172675, 487401505, 470493704, 738534926, 773272596, 420885018,
      437398307, 0, 0, 0, 873080585, 839652098, 671881988, 487402252, 572467239, 621481735, 655565083, 637809170, 302125832, 0, 0, 0};
  alignas(16) static constexpr uint32_t kTc[512] = {
      20352002, 467062190, 480296383, 75986385, 104949229, 115456106, 559428107, 179478071, 203617860, 208236739, 652432713, 246652534, 288001667, 721074862, 369459502, 369459552,
      440832408, 458671128, 40932791, 107446719, 118599169, 129511537, 134347902, 180914721, 644036164, 226713192, 262386920, 279262875, 369405208, 369459552, 369459552, 369459552,
      443875742, 450273703, 56030652, 78709815, 117542992, 145880586, 157854862, 170030236, 613598780, 640242873, 655999599, 283790967, 369459904, 369459552, 369459552, 369459552,
      16781314, 492872724, 76619226, 125939192, 144842257, 178426006, 639201464, 648653008, 669220465, 253369989, 699030772, 728408738, 369459552, 369459552, 369459552, 369459552,
      454362135, 51832860, 483866057, 493937102, 543682658, 131608072, 160982145, 186189994, 670267594, 681819776, 695881976, 732610834, 369459552, 369459552, 369459552, 369459552,
      435160471, 25176074, 44081598, 477567021, 505481281, 561509459, 602448015, 193121454, 213066938, 663334099, 271823084, 369824042, 369459552, 369459552, 369459552, 369459552,
      445659553, 45542839, 337713200, 89213006, 136446063, 583570572, 190371378, 212421813, 257565921, 728472229, 744790307, 369459552, 369459552, 369459552, 369459552, 369459552,
      23088133, 337721048, 88582225, 110207066, 138537482, 176329880, 670666330, 689585398, 699664638, 736809239, 369409733, 369459552, 369459552, 369459552, 369459552, 369459552,
      16151961, 459720721, 498135089, 515349573, 540541018, 561108080, 158904870, 613999156, 651768394, 706371804, 369459485, 369459552, 369459552, 369459552, 369459552, 369459552,
      31893923, 60242975, 520578108, 141058547, 344506923, 660185275, 259236064, 272889490, 286540040, 733659818, 369459914, 369459552, 369459552, 369459552, 369459552, 369459552,
      8389632, 461386144, 482390054, 106000458, 571611665, 599949471, 773012676, 250213707, 271838862, 315925181, 369459552, 369459552, 369459552, 369459552, 369459552, 369459552,
      48697362, 536299980, 663304781, 369412374, 451314079, 530675177, 565303397, 601003561, 641937985, 656622798, 254002397, 274354833, 311091477, 369410350, 369459552, 369459552,
      39881739, 66530757, 509055043, 145847789, 344087701, 209282234, 245704910, 694834428, 312135942, 369412399, 6652256, 101764122, 164774419, 624082089, 703844542, 369459552,
      43014871, 67589167, 521646554, 528997470, 171082885, 667532460, 270162159, 298484377, 313818398, 472306376, 555850236, 594693260, 348337760, 369400474, 369459552, 369459552,
      486595590, 522698209, 612961409, 629750967, 227117665, 690612448, 283383038, 351973710, 739542705, 456549095, 116895188, 574128660, 641256997, 320109205, 369459552, 369459552,
      455095713, 514302395, 551013467, 176319610, 210334908, 242976981, 678671593, 284855539, 726948115, 11957948, 29802514, 546829813, 632875146, 275380438, 369819302, 369459552,
      34629035, 66112549, 539065831, 560480784, 599313556, 206747815, 772375134, 680128101, 778718863, 30841184, 767669282, 566780429, 187225233, 659147345, 315290889, 369459552,
      473367559, 79755316, 99078236, 597157366, 647560765, 659148400, 264487542, 714776223, 745829037, 30844256, 144208939, 650869908, 677615223, 293863674, 742681881, 369459552,
      446708123, 54556699, 114804821, 159524367, 618844739, 205717695, 226079326, 284435101, 738913553, 56033632, 552718424, 136445054, 237573256, 705328782, 737853093, 369459552,
      447750151, 506944974, 563629155, 604141714, 628293196, 229861978, 703214211, 296400613, 369827099, 27683168, 509673526, 109152343, 161003015, 236116127, 723774691, 369459895,
      470219194, 78707145, 544318974, 585250312, 599320111, 196684979, 660191420, 707007114, 369399060, 32934240, 508629031, 574953563, 191025325, 672790111, 271194756, 369459467,
      57093571, 86058045, 122801659, 591960199, 644023874, 305832557, 9797939, 34629039, 518743512, 560067290, 149454558, 230248602, 681190011, 700701941, 727369997, 369459909,
      466002330, 502744522, 588341734, 685387343, 280659609, 296398503, 432374050, 521622584, 535523035, 342369795, 187237507, 645483089, 237734099, 702800110, 731616525, 369459552,
      37785005, 73449926, 520424534, 603053170, 207166022, 261762660, 293251753, 314877630, 74507296, 543248460, 588818563, 239703638, 685477094, 741002493, 369459907, 369459552,
      44061699, 340245570, 578321950, 629752382, 663972049, 270141155, 10164516, 462870946, 506533328, 593653849, 179477048, 234054857, 261755516, 289681673, 369459493, 369459552,
      448807948, 504425516, 126994511, 169396778, 220823112, 294883548, 452228787, 52475936, 84365775, 609380455, 203611312, 225029320, 279190784, 353027344, 369459552, 369459552,
      70305815, 551652830, 138538104, 168327495, 623033507, 716849804, 453284128, 71767490, 338765896, 124898805, 585253410, 218302023, 302228697, 319072546, 369459552, 369459552,
      490135980, 501705789, 526468175, 185111035, 232367709, 247071354, 4908287, 462437797, 101175773, 341316090, 573707382, 165828135, 238633530, 748935410, 369459552, 369459552,
      91692444, 542642690, 579367645, 618212938, 240341589, 281279728, 310045367, 369459907, 36099481, 490162234, 535907808, 586708485, 346239149, 696926853, 746888467, 369459552,
      474416549, 101164488, 113354855, 170440224, 772369593, 776173775, 741011733, 369459505, 28328350, 499183048, 529628639, 174643733, 663956672, 709107356, 352630049, 369459552,
      499163543, 538444260, 565733492, 152190088, 628686994, 241376857, 709495018, 369459884, 335549440, 61249549, 81234393, 527937614, 579990034, 627645604, 711183987, 369459552,
      492877528, 90677720, 340898286, 557966862, 162680135, 776163924, 748356895, 369459552, 21392387, 38195221, 148400225, 198354480, 207817918, 673401447, 322643640, 369459552};
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
  static constexpr int kMaxRkck = 32;
  static constexpr int kMaxRkc = 2;
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
      0, 1, 2, 3, 4, 5, 6, 7, 9, 10, 11, 12, 13, 14, 15, 16,
      17, 18, 19, 20, 21, 22, 23, 24, 26, 27, 28, 29, 30, 31, 32, 33,
      34, 35, 36, 37, 38, 39, 40, 41, 42, 43, 44, 45, 46, 47, 48, 49,
      50, 51, 52, 53, 54, 55, 56, 57, 58, 59, 60, 61, 62, 63, 64, 65,
      66, 67, 68, 69, 70, 71, 72, 73, 74, 75, 76, 77, 78, 79, 81, 82,
      83, 84, 85, 86, 87, 88, 89, 90, 91, 93, 94, 95, 96, 97, 98, 99,
      100, 101, 102, 103, 105, 106, 107, 108, 109, 110, 111, 112, 113, 114, 115, 116,
      117, 118, 119, 120, 121, 124, 125, 126, 127, 128, 129, 130, 131, 132, 133, 134,
      135, 136, 137, 138, 139, 140, 141, 143, 144, 145, 146, 147, 148, 149, 150, 151,
      152, 153, 154, 155, 156, 157, 158, 159, 160, 161, 163, 164, 165, 166, 167, 168,
      169, 170, 171, 172, 173, 174, 175, 176, 177, 178, 179, 180, 181, 182, 183, 184,
      185, 186, 187, 188, 189, 190, 191, 192, 193, 194, 195, 196, 197, 198, 199, 200,
      201, 202, 203, 204, 205, 206, 207, 208, 209, 210, 211, 212, 213, 214, 216, 217,
      218, 219, 220, 221, 222, 223, 224, 225, 226, 227, 228, 229, 230, 232, 233, 234,
      236, 237, 238, 239, 240, 241, 242, 243, 244, 246, 247, 248, 249, 250, 251, 252,
      253, 254, 255, 256, 257, 258, 259, 260, 261, 262, 263, 264, 265, 266, 267, 268,
      269, 270, 271, 272, 273, 274, 275, 277, 278, 279, 280, 281, 282, 283, 284, 285,
      286, 287, 289, 290, 291, 292, 293, 294, 296, 297, 298, 299, 300, 301, 302, 303,
      304, 305, 306, 307, 308, 309, 310, 311, 312, 313, 314, 315, 316, 317, 318, 319,
      320, 321, 323, 324, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1,
      8, 25, 80, 92, 104, 122, 123, 142, 162, 215, 231, 235, 245, 276, 288, 295,
      322, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1,
      -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1,
      -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1, -1};
  // LDS byte offsets within the system's area: each lane's rate operands
  // (R x 4), and the signed rates of its species in reaction order
  alignas(16) static constexpr uint16_t kOp[1536] = {
      128, 384, 56, 248, 88, 184, 144, 272, 72, 128, 64, 104, 88, 384, 296, 320,
      152, 184, 0, 240, 144, 424, 56, 112, 104, 208, 128, 248, 16, 344, 112, 128,
      336, 416, 176, 184, 176, 408, 24, 392, 72, 360, 144, 408, 16, 200, 184, 424,
      72, 360, 152, 264, 56, 416, 128, 408, 88, 184, 64, 232, 384, 400, 0, 264,
      136, 144, 80, 200, 344, 424, 64, 200, 136, 272, 40, 408, 144, 152, 168, 400,
      40, 384, 8, 120, 88, 200, 40, 264, 152, 328, 128, 248, 344, 424, 24, 288,
      40, 296, 152, 224, 32, 72, 24, 80, 192, 384, 168, 200, 256, 368, 248, 296,
      104, 200, 160, 416, 8, 8, 408, 424, 8, 304, 56, 200, 320, 384, 72, 312,
      304, 336, 144, 224, 152, 264, 96, 288, 320, 344, 176, 192, 336, 424, 16, 224,
      72, 256, 176, 352, 224, 264, 64, 288, 240, 360, 248, 416, 32, 280, 40, 264,
      232, 296, 256, 400, 304, 424, 8, 80, 112, 320, 88, 216, 32, 168, 120, 152,
      168, 408, 152, 392, 96, 296, 384, 400, 8, 88, 0, 320, 344, 424, 16, 168,
      128, 192, 88, 248, 136, 320, 24, 264, 344, 408, 232, 384, 80, 376, 0, 280,
      216, 352, 296, 416, 240, 424, 400, 416, 192, 248, 312, 344, 104, 360, 152, 392,
      208, 368, 240, 296, 96, 328, 128, 312, 144, 232, 312, 336, 96, 368, 264, 424,
      64, 280, 128, 128, 176, 376, 24, 248, 104, 248, 152, 256, 152, 176, 64, 184,
      72, 136, 0, 104, 248, 424, 360, 400, 80, 312, 256, 400, 56, 128, 112, 160,
      24, 104, 112, 400, 112, 176, 128, 320, 152, 160, 80, 136, 8, 280, 248, 424,
      264, 416, 248, 376, 88, 312, 120, 216, 208, 224, 64, 328, 200, 208, 192, 360,
      264, 280, 304, 312, 120, 408, 328, 424, 104, 104, 56, 280, 384, 400, 56, 200,
      32, 80, 40, 160, 192, 288, 104, 328, 320, 384, 8, 344, 16, 368, 104, 424,
      224, 368, 64, 296, 80, 400, 56, 64, 64, 208, 112, 344, 96, 120, 192, 400,
      64, 232, 112, 176, 8, 88, 176, 424, 56, 336, 72, 224, 136, 272, 32, 376,
      72, 392, 128, 384, 104, 392, 248, 368, 56, 256, 280, 296, 64, 96, 176, 424,
      112, 112, 152, 320, 72, 96, 0, 112, 224, 408, 24, 352, 8, 40, 24, 152,
      136, 216, 0, 416, 176, 424, 0, 320, 112, 136, 72, 376, 16, 280, 32, 200,
      128, 304, 336, 384, 104, 416, 192, 408, 152, 392, 296, 416, 0, 0, 0, 0,
      64, 240, 48, 256, 192, 368, 64, 392, 56, 192, 88, 384, 32, 216, 40, 376,
      216, 288, 184, 264, 0, 0, 0, 0, 296, 416, 200, 264, 200, 280, 128, 360,
      120, 376, 16, 328, 152, 152, 8, 128, 288, 416, 280, 360, 0, 0, 0, 0,
      88, 96, 40, 152, 72, 208, 120, 200, 112, 416, 96, 240, 0, 128, 16, 304,
      136, 168, 160, 312, 0, 0, 0, 0, 32, 376, 40, 408, 56, 144, 64, 296,
      64, 72, 224, 400, 240, 296, 264, 280, 176, 384, 192, 368, 0, 0, 0, 0,
      112, 288, 144, 200, 264, 400, 16, 288, 272, 368, 112, 152, 72, 392, 0, 256,
      88, 216, 48, 280, 0, 0, 0, 0, 192, 264, 168, 184, 16, 344, 272, 304,
      24, 160, 72, 400, 160, 264, 104, 296, 264, 264, 200, 288, 0, 0, 0, 0,
      0, 344, 104, 128, 176, 408, 136, 232, 160, 360, 200, 296, 112, 144, 104, 176,
      232, 264, 104, 240, 0, 0, 0, 0, 24, 256, 96, 344, 288, 416, 264, 312,
      40, 416, 184, 272, 112, 216, 24, 312, 184, 416, 240, 376, 0, 0, 0, 0,
      104, 184, 272, 352, 8, 144, 72, 200, 120, 136, 0, 344, 112, 152, 88, 408,
      0, 176, 88, 136, 0, 0, 0, 0, 72, 280, 296, 320, 176, 296, 80, 280,
      64, 376, 16, 280, 192, 336, 88, 344, 272, 344, 88, 240, 0, 0, 0, 0,
      208, 264, 184, 256, 280, 416, 216, 248, 96, 208, 112, 312, 56, 216, 72, 376,
      120, 376, 144, 216, 0, 0, 0, 0, 40, 328, 240, 336, 216, 224, 192, 400,
      72, 392, 112, 352, 216, 336, 32, 192, 200, 400, 72, 376, 0, 0, 0, 0,
      104, 360, 296, 416, 24, 256, 144, 216, 64, 336, 88, 224, 160, 416, 184, 368,
      280, 344, 144, 208, 0, 0, 0, 0, 72, 312, 80, 416, 32, 216, 96, 320,
      312, 320, 248, 272, 216, 264, 152, 312, 64, 152, 16, 144, 0, 0, 0, 0,
      64, 104, 0, 120, 56, 144, 224, 368, 264, 328, 168, 248, 112, 240, 176, 416,
      272, 304, 24, 168, 0, 0, 0, 0, 32, 248, 96, 344, 144, 152, 40, 352,
      72, 312, 144, 376, 48, 128, 64, 272, 40, 192, 176, 320, 0, 0, 0, 0,
      224, 312, 336, 360, 216, 320, 184, 272, 160, 216, 112, 368, 320, 408, 8, 232,
      8, 32, 24, 136, 0, 0, 0, 0, 160, 184, 288, 400, 192, 224, 88, 168,
      224, 256, 144, 168, 32, 176, 224, 272, 184, 304, 64, 392, 0, 0, 0, 0,
      64, 280, 40, 288, 32, 392, 112, 264, 96, 160, 56, 152, 96, 344, 120, 376,
      296, 416, 168, 408, 0, 0, 0, 0, 112, 136, 96, 104, 184, 328, 192, 248,
      112, 248, 192, 200, 144, 312, 240, 304, 280, 368, 160, 312, 0, 0, 0, 0,
      112, 264, 248, 400, 128, 256, 104, 328, 192, 216, 312, 320, 80, 248, 120, 384,
      248, 336, 64, 328, 0, 0, 0, 0, 128, 160, 80, 104, 8, 160, 0, 368,
      128, 408, 96, 264, 152, 256, 264, 280, 200, 288, 304, 360, 0, 0, 0, 0,
      104, 264, 128, 384, 48, 360, 200, 272, 216, 288, 200, 280, 184, 200, 104, 416,
      232, 256, 192, 248, 0, 0, 0, 0, 160, 232, 144, 152, 72, 384, 160, 200,
      88, 384, 40, 352, 32, 184, 24, 280, 112, 296, 288, 400, 0, 0, 0, 0,
      216, 368, 128, 408, 104, 384, 264, 368, 8, 192, 152, 184, 80, 408, 384, 400,
      16, 176, 24, 128, 0, 0, 0, 0, 24, 328, 64, 240, 96, 304, 104, 152,
      184, 392, 264, 312, 40, 384, 32, 264, 120, 368, 104, 144, 0, 0, 0, 0,
      216, 392, 248, 376, 8, 72, 16, 368, 176, 296, 104, 144, 88, 264, 128, 128,
      120, 304, 288, 336, 0, 0, 0, 0, 48, 368, 16, 128, 224, 304, 296, 336,
      104, 264, 80, 360, 80, 312, 104, 280, 128, 240, 248, 320, 0, 0, 0, 0,
      24, 400, 0, 48, 304, 360, 264, 264, 0, 232, 96, 128, 152, 360, 8, 248,
      200, 344, 192, 264, 0, 0, 0, 0, 128, 288, 144, 264, 120, 184, 64, 208,
      288, 288, 168, 352, 80, 240, 144, 184, 64, 408, 200, 400, 0, 0, 0, 0,
      128, 304, 64, 288, 160, 272, 72, 112, 24, 56, 0, 32, 152, 280, 216, 304,
      88, 216, 24, 192, 0, 0, 0, 0, 320, 368, 72, 184, 160, 184, 104, 104,
      176, 376, 112, 184, 96, 344, 152, 192, 144, 360, 208, 368, 0, 0, 0, 0,
      160, 184, 0, 168, 8, 256, 288, 376, 72, 112, 8, 336, 64, 344, 192, 224,
      16, 40, 48, 400, 0, 0, 0, 0, 136, 264, 96, 352, 112, 200, 24, 392,
      72, 304, 128, 160, 160, 184, 56, 280, 224, 416, 40, 392, 0, 0, 0, 0,
      392, 400, 216, 296, 184, 264, 232, 384, 160, 304, 80, 296, 136, 288, 152, 352,
      0, 0, 0, 0, 0, 0, 0, 0, 48, 248, 112, 232, 104, 264, 72, 392,
      72, 88, 64, 64, 88, 168, 64, 344, 0, 0, 0, 0, 0, 0, 0, 0,
      184, 184, 272, 392, 280, 336, 192, 224, 48, 304, 80, 272, 120, 136, 200, 224,
      0, 0, 0, 0, 0, 0, 0, 0, 88, 184, 112, 176, 16, 168, 24, 288,
      48, 296, 0, 176, 232, 248, 344, 416, 0, 0, 0, 0, 0, 0, 0, 0,
      0, 416, 8, 184, 232, 296, 152, 168, 136, 176, 128, 152, 96, 200, 8, 184,
      0, 0, 0, 0, 0, 0, 0, 0, 176, 312, 120, 416, 96, 96, 16, 376,
      224, 408, 112, 368, 168, 360, 288, 312, 0, 0, 0, 0, 0, 0, 0, 0,
      136, 264, 56, 360, 152, 248, 200, 280, 8, 336, 128, 400, 192, 200, 104, 240,
      0, 0, 0, 0, 0, 0, 0, 0, 48, 360, 320, 376, 56, 328, 104, 168,
      8, 168, 160, 416, 176, 416, 248, 272, 0, 0, 0, 0, 0, 0, 0, 0,
      32, 360, 72, 416, 88, 352, 56, 344, 64, 352, 160, 280, 96, 112, 216, 400,
      0, 0, 0, 0, 0, 0, 0, 0, 0, 208, 32, 392, 16, 208, 112, 184,
      16, 344, 40, 264, 184, 192, 120, 416, 0, 0, 0, 0, 0, 0, 0, 0,
      8, 144, 160, 216, 264, 320, 104, 232, 112, 304, 40, 352, 208, 400, 176, 200,
      0, 0, 0, 0, 0, 0, 0, 0, 16, 152, 96, 400, 96, 344, 104, 232,
      56, 120, 88, 296, 144, 400, 32, 304, 0, 0, 0, 0, 0, 0, 0, 0};
  alignas(16) static constexpr uint16_t kTm[2816] = {
      4224, 704, 816, 848, 4480, 4520, 1088, 1272, 1680, 5424, 1856, 1912, 2000, 2048, 5728, 2160,
      2496, 2552, 2576, 2624, 6288, 3136, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4072, 896, 4528, 4752,
      6624, 6624, 4856, 4896, 4944, 3056, 1496, 5392, 1872, 5520, 5528, 5696, 2136, 6680, 2256, 2352,
      2432, 6136, 2600, 6704, 6352, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6600, 808, 4536, 4552, 4680, 1136, 4728, 1312,
      3048, 4984, 1416, 5032, 3064, 1624, 1688, 5544, 2144, 6696, 2744, 6416, 6480, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 4232, 4376, 4400, 992, 1024, 1040, 3032, 4784, 1368, 1400, 5144, 1600,
      5240, 5440, 1992, 2112, 2184, 2312, 2752, 2768, 2832, 2880, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4200, 4296, 4512, 936, 4576, 4600, 1080, 1096, 4792, 4832, 5160, 1856, 5616, 5712, 2216, 5848,
      5896, 2328, 2488, 6352, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 472, 4064, 608, 616,
      4264, 736, 1224, 5080, 1576, 5256, 1800, 1960, 1968, 2008, 2032, 5696, 2128, 5912, 6344, 6480,
      2904, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 592, 4392, 816, 4456, 4504, 4864, 5488, 5496,
      5832, 2672, 2896, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 448, 488, 3008, 552, 4152, 912, 4560, 4632, 1064, 1072, 4712, 4800,
      5016, 1440, 5200, 1760, 5440, 5560, 5792, 2392, 6200, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4112, 560, 4176, 4288, 4320, 792, 832, 1008, 3024, 1072, 1104, 1128, 1336, 1472, 1488, 1568,
      5168, 5224, 5272, 5296, 1896, 1896, 5536, 2064, 2248, 5968, 2408, 6192, 6712, 6328, 2776, 2800,
      6456, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4048, 4080, 568, 584,
      4248, 4280, 840, 928, 4576, 1000, 4672, 4704, 1168, 4872, 4896, 1344, 1384, 5056, 5176, 5224,
      1656, 5288, 5320, 5456, 5464, 5480, 5744, 2208, 6088, 6160, 2728, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4120, 696, 760, 992, 4656, 1176, 3056, 5160,
      1832, 1888, 1904, 5632, 5872, 5904, 5928, 5944, 2512, 2584, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 504, 512, 4192, 4472, 4544, 4640, 1240, 5024, 5072, 1616, 1712, 5384,
      5480, 1976, 5568, 5592, 2192, 2200, 5920, 5992, 6136, 6704, 6256, 2704, 2712, 6464, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4192, 648, 712, 744, 856, 952, 4672, 1208, 4888, 5000, 5000, 5048, 1632, 5280, 5344, 1784,
      1840, 2024, 5624, 5640, 6664, 5680, 5856, 5960, 6016, 6048, 6712, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4040, 4136, 4136, 640,
      4240, 4272, 4288, 744, 760, 4352, 4616, 1264, 4880, 1304, 1352, 1352, 4968, 1432, 1456, 1464,
      1472, 5136, 5144, 1824, 5416, 2088, 5688, 5704, 2168, 2176, 2304, 2344, 2448, 6112, 3112, 2576,
      2688, 2840, 3520, 3520, 3520, 3520, 3520, 3520, 4088, 3008, 4160, 4160, 4168, 4208, 4328, 4336,
      872, 888, 968, 1048, 1088, 1248, 1344, 4952, 1448, 1560, 1584, 5216, 1648, 1696, 1704, 1744,
      5352, 1864, 5456, 1928, 5552, 5656, 5760, 5768, 5776, 5824, 6048, 2608, 6408, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 704, 904, 1016, 1056, 1120, 4920, 1496, 5208, 5264, 5560, 5680, 2272,
      2288, 6688, 6000, 2472, 6304, 6424, 6432, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4032, 456, 4096, 528, 528, 640, 4344, 768, 784, 808, 4408, 4416, 968, 976, 4632, 1112,
      4848, 5056, 1592, 5192, 5368, 1840, 1880, 1920, 1936, 2056, 2072, 2136, 5728, 5832, 2336, 2336,
      2520, 2832, 6440, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4056, 4168, 4328, 4440,
      4496, 4608, 4664, 1152, 5264, 5504, 5984, 6000, 6096, 6160, 2584, 6208, 6240, 2704, 2768, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 6592, 624, 776, 824, 4528, 960, 4568, 4712,
      4752, 1200, 4800, 4808, 1512, 1736, 1752, 1824, 5760, 5864, 2360, 6072, 2504, 6096, 6152, 2720,
      2736, 2744, 2840, 6472, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 464, 480, 576, 608, 776, 4536, 4568, 1016, 1032, 4808, 1304, 1408,
      5008, 1528, 1552, 1648, 1760, 1808, 1920, 5608, 5648, 2112, 5720, 5720, 5776, 2232, 5880, 5936,
      5952, 2376, 2400, 6080, 6104, 6168, 6216, 6328, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4312, 4344, 4360, 4432, 944, 1048, 4856, 1288, 4928, 4936, 1576, 5240, 5248, 5328, 5344, 1880,
      5472, 1944, 1952, 5752, 5808, 5976, 2528, 6168, 2656, 2792, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 632, 848, 984, 4600,
      1240, 4984, 1408, 1432, 1504, 3064, 5112, 1728, 1752, 1848, 5528, 5992, 6024, 6240, 2752, 2784,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 496, 888, 4488, 4624, 4736, 4760, 1480, 5408,
      5448, 1912, 5504, 5576, 5648, 5656, 2176, 2240, 5848, 6040, 2480, 2536, 2608, 3120, 6248, 3128,
      6288, 2760, 6416, 6720, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 632, 3016, 4240, 672, 4312, 840, 4432, 4464, 4464, 4472, 896, 4544,
      1232, 4840, 4920, 4936, 4960, 1448, 1480, 5072, 1672, 1808, 5400, 1864, 2064, 2224, 5888, 5896,
      2360, 5976, 2432, 6056, 6080, 2640, 6280, 6360, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4096, 4104, 4216, 4688, 1192, 4824, 1256, 1392, 5088, 5200, 1768, 5360, 5392, 2080, 5672, 2096,
      2120, 5784, 2216, 2376, 2384, 6032, 6056, 2536, 2664, 6344, 2816, 2864, 2880, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 488, 600, 624, 6600,
      1064, 3024, 1096, 4696, 1120, 1168, 1280, 1288, 4952, 1424, 1504, 1664, 1768, 1792, 5592, 5664,
      5888, 2416, 6016, 6032, 2480, 2512, 6112, 2680, 6312, 6392, 6448, 2872, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4040, 4256, 4520, 4704, 1336, 5032, 5128, 5152,
      5168, 5280, 5664, 6064, 2736, 2888, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 504, 4368, 4384, 864, 944, 1056, 1184, 4776, 1200, 4792, 4816, 5328,
      5360, 5376, 5712, 5768, 5792, 5800, 5816, 2368, 2464, 6144, 6208, 6224, 6256, 2720, 6464, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      480, 4144, 568, 4304, 4592, 4776, 1216, 4824, 4904, 3048, 1392, 1512, 5152, 5184, 1640, 1712,
      5336, 5512, 2264, 2384, 2416, 6488, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4360, 872, 1152, 1376,
      4992, 1456, 1464, 1488, 1536, 5424, 2256, 6008, 6128, 6152, 6192, 6272, 6400, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4176, 680, 792, 5104, 1544, 1632, 6656, 5736,
      5824, 2280, 5944, 2448, 2496, 2688, 2696, 2712, 6440, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 448, 456, 512, 4104, 544, 4296, 752, 800, 4456, 1040, 1184, 1256,
      5008, 1520, 5136, 1720, 1728, 5352, 2016, 2104, 6672, 3096, 5872, 2352, 6008, 2456, 2520, 6384,
      2816, 2856, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4080, 536, 592, 4232, 672, 4784, 4848, 4944, 1552, 5336, 5600, 2160, 5880, 2544, 6200, 6400,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 464, 4128, 600, 4216,
      4256, 4336, 4352, 824, 4440, 4496, 4592, 1024, 4720, 1160, 1248, 1296, 1328, 1328, 4960, 4968,
      5040, 5312, 1784, 1816, 5416, 1960, 2000, 2008, 5608, 2032, 3080, 2152, 5752, 5816, 2296, 2328,
      5920, 6176, 2640, 6264, 6264, 6272, 2864, 3520, 4056, 656, 880, 960, 4664, 1144, 1232, 1280,
      4928, 5232, 1672, 1720, 1904, 2248, 2264, 2456, 6296, 6336, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 4112, 552, 4248, 4320, 4680, 4696, 1176, 4768, 4976, 1424, 1688, 1792,
      1952, 5616, 2048, 2152, 6680, 2296, 2312, 2344, 5952, 2392, 6176, 2616, 2648, 2672, 6320, 6376,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4208, 728, 736, 4408, 832, 1008, 1136, 3032, 4744, 1360, 1400, 5376, 5432, 5432, 2024, 5672,
      5984, 2440, 6224, 6232, 2680, 6392, 2824, 2848, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4064, 560, 4184, 664,
      688, 864, 1128, 4760, 1320, 4992, 1544, 1664, 5408, 1888, 5496, 1976, 1984, 2016, 5624, 5736,
      2168, 6128, 2560, 2616, 2632, 6368, 6408, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4072, 4416, 1144, 4888, 4904, 4912, 6640, 5096,
      5192, 5464, 5472, 5488, 5552, 2144, 2280, 2368, 2488, 2592, 6336, 6360, 2808, 6432, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 520, 4120, 4280, 4304, 4488, 1000, 4640, 1160, 1696, 5304, 5320, 1776,
      1816, 2056, 2184, 2232, 5864, 5928, 2440, 2568, 2592, 2656, 2792, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4088, 576, 664, 4424, 920, 4584, 4608, 1208, 4816, 5040, 5304, 1776, 1984, 2072, 5840, 6120,
      2552, 6184, 2760, 2856, 3136, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4264, 4376, 4840, 1264,
      5016, 1568, 1624, 5312, 5640, 2088, 3104, 6104, 2800, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4152, 680, 720, 1320, 6632, 4976, 5064, 5096,
      1608, 5296, 1872, 5520, 5784, 5800, 2568, 6384, 2848, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 520, 4224, 648, 712, 4552, 6608, 4728, 6616, 1440, 5048, 6648, 5120,
      1584, 1680, 5544, 2200, 5856, 5960, 5968, 2408, 2424, 6120, 2600, 6296, 6320, 6448, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      496, 656, 856, 1224, 5024, 1600, 1704, 1800, 1848, 5536, 1968, 2400, 6144, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4048, 4272, 720, 912,
      4504, 4512, 4616, 1112, 4864, 4912, 5104, 5248, 1832, 2080, 3088, 5936, 6024, 6088, 2648, 2808,
      6472, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4144, 4368, 4392, 4424, 4688, 1216, 1272, 1296,
      1312, 5128, 5232, 1744, 1928, 5600, 6664, 2104, 2224, 6696, 2664, 6376, 6424, 2888, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 544, 584, 4200, 800, 920, 4624, 1080, 1360, 1416, 5208, 5272, 1736,
      5448, 5632, 2128, 2208, 2272, 2696, 6304, 2728, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4032, 768, 4584, 4648, 4872, 4880, 1376, 5080, 5088, 1536, 1592, 1608, 1616, 5384, 5568, 5584,
      2040, 2288, 2320, 5912, 6184, 6248, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 4384, 4448, 880, 936,
      1032, 1104, 4832, 1368, 1384, 1528, 5176, 5288, 5400, 1992, 5688, 5744, 6216, 2776, 2904, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 536, 728, 752, 4400, 4448, 952, 984, 4648,
      4656, 4720, 1192, 1560, 1640, 1656, 3072, 1936, 5584, 2040, 2096, 3088, 2320, 2464, 6064, 6072,
      2544, 6312, 2824, 2872, 2896, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 472, 616, 784, 976, 4736, 3040, 5112, 5120, 5184, 5368, 5512, 5576,
      2120, 2192, 5840, 6688, 5904, 2504, 2784, 6456, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520, 3520,
      4128, 4184, 688, 696, 4480, 904, 928, 4560, 4744, 4768, 5064, 1520, 5216, 5256, 3072, 1944,
      5704, 5808, 2240, 2304, 2424, 6040, 2472, 2528, 2560, 2624, 2632, 6232, 6280, 6368, 6488, 3520,
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
