// rk_pleiades.hip -- the Pleiades problem (Sec. 4.1): seven bodies of mass
// m_i = i moving in the plane under their mutual gravitation, as 28
// first-order equations (z, w)' = (w, f(z)) with z = (x_1..x_7, y_1..y_7):
//   x_i'' = sum_{j != i} m_j (x_j - x_i) / r_ij,   y_i'' likewise,
//   r_ij = ((x_i - x_j)^2 + (y_i - y_j)^2)^(3/2)   (the y difference squared);
// no per-system parameters.  r_ij^(3/2) is formed as d2 sqrt(d2) and the
// division by it as a multiplication by its reciprocal, once per pair (the
// pair's value is the same bits for (i, j) and (j, i): the squared differences
// of negated operands are equal).  Each body's sums run over j in increasing
// order from zero.  Its 28-vectors are too many for registers in the RKCK
// driver: one lane per system keeps them in workspace columns (the column
// tier, plain and persistent schedules), and the group variant spreads a
// system over eight lanes (the group schedule, the default).
#include "rk_launch.hpp"
#include "rk_group.hpp"

namespace rkmi {

struct PleiadesProblem {
  static constexpr int N = 28;
  static constexpr bool kColumns = true;
  static constexpr int kGroupLanes = 1;
  static constexpr int kLaneDoubles = 0;
  using Params = const double*;
  struct Lane {};
  RKMI_HD static void init(Lane&, const Params&, const double* __restrict__, int64_t, int64_t,
                           double*) {}
  template <class VI, class VO>
  RKMI_HD static void rhs(const Lane&, const Params&, const VI& y, VO& f) {
    double x[7], yy[7], rinv[7][7];
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      x[i] = y[i];
      yy[i] = y[7 + i];
    }
#pragma unroll
    for (int i = 0; i < 14; ++i) f[i] = y[14 + i];
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
      for (int j = i + 1; j < 7; ++j) {
        const double d2 = (x[i] - x[j]) * (x[i] - x[j]) + (yy[i] - yy[j]) * (yy[i] - yy[j]);
        rinv[i][j] = 1.0 / (d2 * sqrt(d2));
        rinv[j][i] = rinv[i][j];
      }
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      double ax = 0.0, ay = 0.0;
#pragma unroll
      for (int j = 0; j < 7; ++j) {
        if (j == i) continue;
        const double mj = (double)(j + 1);
        ax += (mj * (x[j] - x[i])) * rinv[i][j];
        ay += (mj * (yy[j] - yy[i])) * rinv[i][j];
      }
      f[14 + i] = ax;
      f[21 + i] = ay;
    }
  }
};

// Group variant: lane r < 7 of a group of eight holds body r's unknowns
// (x_r, y_r, x_r', y_r') in registers; lane 7 holds none.  An evaluation
// writes the positions to the group's LDS area; the 21 pair values
// 1 / (d2 sqrt(d2)) are formed once each, three per lane (pair p by lane p mod
// 7, with the smaller body index first as the one-lane code forms them), and
// stored for both orders; each body's lane then sums its terms in the one-lane
// order, so results equal the one-lane kernels.
//
// Bound: VALU issue (a square root and a division per pair).  Nothing branches:
// a body's own term is (x_i - x_i) times a zero kept on the diagonal, which adds
// +-0 to a sum that is never -0, and lane 7 repeats pairs of lanes 0..2 without a
// body to sum for.  Positions lie as (x, y) and the pair values of a body in
// rows of ten doubles, so all reads are of 16 bytes and the rows of a group's
// lanes meet in no bank.  With a branch around each body's own term and reads of
// single doubles, RKCK over ten steps took 19.9 ms at 262144 systems and 1.35 ms
// at 2001, where now 18.9 and 1.03; RKC at 2001 systems 103, now 92.
constexpr int kPleiadesRow = 10;   // doubles of a body's row of pair values
// Pair p of the bodies a < b (p = 21: pair 0 again, for lane 7): the places of
// their positions and of the pair's value in a group's area.
struct PleiadesPairs {
  int16_t a[22], b[22];
  constexpr PleiadesPairs() : a(), b() {
    int p = 0;
    for (int i = 0; i < 7; ++i)
      for (int j = i + 1; j < 7; ++j) {
        a[p] = (int16_t)i;
        b[p] = (int16_t)j;
        ++p;
      }
    a[21] = a[0];
    b[21] = b[0];
  }
};
inline constexpr PleiadesPairs kPleiadesPairs{};

struct PleiadesGroup {
  static constexpr int N = 28;
  static constexpr int NR = 0;
  static constexpr int kL = 8;
  static constexpr int kGroupLanes = 8;
  static constexpr bool kColumns = false;
  static constexpr int kLaneDoubles = 0;
  static constexpr int S = 4;
  // RKCK fits three waves per SIMD (four spill: 20.1 ms at 262144 systems); RKC
  // two with a few spills (9000 systems: 122 ms, one wave 166)
  static constexpr int kWavesPerEuRkck = 3;
  static constexpr int kWavesPerEuRkc = 2;
  static constexpr bool kOwnRhs = true;
  static constexpr int kOffPos = 0;                            // (x_i, y_i), lane 7's place
  static constexpr int kOffPair = 16;                          // 1 / r_ij at i kPleiadesRow + j
  static constexpr int kOffRed = kOffPair + 8 * kPleiadesRow;  // norm scratch, N doubles
  static constexpr int kLdsPerSystem = kOffRed + N;
  static constexpr int kSp[S * kL] = {0,  1,  2,  3,  4,  5,  6,  -1,     // x_r
                                      7,  8,  9,  10, 11, 12, 13, -1,     // y_r
                                      14, 15, 16, 17, 18, 19, 20, -1,     // x_r'
                                      21, 22, 23, 24, 25, 26, 27, -1};    // y_r'
  using Params = const double*;
  struct Lane {
    int pa[3], pb[3], va[3], vb[3];   // its pairs' positions and values
  };
  __device__ static void init(Lane& L, const Params&, const double* __restrict__, int64_t,
                              int64_t, const Grp<PleiadesGroup>& x) {
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const int a = kPleiadesPairs.a[x.r + 7 * t], b = kPleiadesPairs.b[x.r + 7 * t];
      L.pa[t] = a;
      L.pb[t] = b;
      L.va[t] = kOffPair + a * kPleiadesRow + b;
      L.vb[t] = kOffPair + b * kPleiadesRow + a;
    }
    x.lds[kOffPair + x.r * (kPleiadesRow + 1)] = 0.0;   // the diagonal
  }
  __device__ static void rhs(const Lane& L, const Grp<PleiadesGroup>& x, const double (&y)[S],
                             double (&f)[S]) {
    double2* const P = reinterpret_cast<double2*>(x.lds + kOffPos);
    P[x.r] = make_double2(y[0], y[1]);
    group_sync();
    double rinv[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const double2 a = P[L.pa[t]], b = P[L.pb[t]];
      const double d2 = (a.x - b.x) * (a.x - b.x) + (a.y - b.y) * (a.y - b.y);
      rinv[t] = 1.0 / (d2 * sqrt(d2));
    }
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      x.lds[L.va[t]] = rinv[t];
      x.lds[L.vb[t]] = rinv[t];
    }
    group_sync();
    const double2* const row =
        reinterpret_cast<const double2*>(x.lds + kOffPair + x.r * kPleiadesRow);
    double ax = 0.0, ay = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double2 r2 = row[q];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int j = 2 * q + h;
        if (j == 7) continue;
        const double2 p = P[j];
        const double mj = (double)(j + 1), rj = h ? r2.y : r2.x;
        ax += (mj * (p.x - y[0])) * rj;
        ay += (mj * (p.y - y[1])) * rj;
      }
    }
    const bool body = x.r < 7;
    f[0] = body ? y[2] : 0.0;
    f[1] = body ? y[3] : 0.0;
    f[2] = body ? ax : 0.0;
    f[3] = body ? ay : 0.0;
    group_sync();
  }
};

}  // namespace rkmi

extern "C" int rkmi_pleiades_launch(const rkmi::LaunchArgs* a, void* s) {
  return rkmi::launch_with_group<rkmi::PleiadesProblem, rkmi::PleiadesGroup>(a, s);
}

extern "C" int rkmi_pleiades_host(const rkmi::LaunchArgs* a) {
  return rkmi::host_run<rkmi::PleiadesProblem>(a);
}

extern "C" int64_t rkmi_pleiades_workspace(int method, int schedule, int64_t n) {
  return rkmi::workspace_with_group<rkmi::PleiadesProblem, rkmi::PleiadesGroup>(method, schedule,
                                                                                n);
}
