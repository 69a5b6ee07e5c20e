// rk_launch.hpp -- host-side launch plumbing shared by every compiled problem.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "rk_device.hpp"
#include "rk_types.hpp"

namespace rkmi {

enum : int { kSchedAuto = 0, kSchedPlain = 1, kSchedPersistent = 2, kSchedGroup = 3 };

// Launch error codes (mapped to RK_* by the ABI layer).
enum : int { kLaunchOk = 0, kLaunchInvalid = -1, kLaunchHip = -3, kLaunchWorkspace = -5 };

// Workspace layout: [queue head, kQueueBytes][column blocks, one per workgroup].
constexpr size_t kQueueBytes = 256;

// Idle lanes that make a wave of the persistent kernel take new systems.
constexpr int kDefaultRefill = 16;

template <int = 0>
__global__ void queue_reset_kernel(unsigned long long* queue) {
  queue[0] = 0ull;
}

// Bytes of column workspace one workgroup uses (zero for register-held systems).
template <class Prob, int Method>
constexpr size_t block_col_bytes() {
  return Prob::kColumns ? (size_t)slot_doubles<Prob, Method>() * kLdsStride * sizeof(double) : 0;
}

// Systems per wave of a one-lane kernel over n systems.  A wave lasts as long as
// its slowest system and runs every branch that one of its systems takes, so a
// small batch is spread over the chip.  The other lanes repeat the wave's systems
// (spread_position): with the mask left partly empty instead, the same waves took
// 1.2x longer alone and 2.2x with one on every SIMD (van der Pol, four systems a
// wave, 1024 waves: 0.91 against 0.36 ms; 64 waves of 64 systems: 0.45 ms).
// Cheap problems take as few systems as still fit one wave on every SIMD (64 beyond
// 63 systems per SIMD; a second wave per SIMD costs more than it spreads: 2048 waves
// of two systems 0.49, 1024 of four 0.36 ms).  Kernels that fill a SIMD's registers
// (whole_simd) leave half of the SIMDs to batches on other streams, which find no
// room beside them otherwise: one to two waves per compute unit, up to 64 systems
// each.  On every SIMD instead, one call alone took 4-11 % less at 9 species RKC with
// 1500 to 30000 systems and as long or up to 19 % longer elsewhere, but four calls at
// once three times as long (ms, one / two / four streams, before any spreading, on
// every SIMD, so): 13 species RKC 4096 systems 11.2 / 15.6 / 16.1, 9.5 / 17.8 / 33.2,
// 9.7 / 10.0 / 10.5; 16384 systems RKCK 1.09 / 1.42 / 1.64, 1.17 / 1.71 / 2.76, 0.98 /
// 1.21 / 1.36; 9 species RKC 4096 systems 30.7 / 40.4 / 42.0, 19.9 / 39.7 / 69.8, 22.2 /
// 23.0 / 23.5; 13 species + T RKC 4096 systems 84 / 98 / 100, 42 / 79 / 148, 43 / 46 / 46.
constexpr int systems_per_wave(int64_t n, int64_t cus, bool whole_simd) {
  const int64_t l = whole_simd ? n / cus : (n + 4 * cus - 1) / (4 * cus);
  return (int)(l < 1 ? 1 : l > kLdsStride ? kLdsStride : l);
}

// The same on the current device; a problem compiled for a stated number of waves
// per SIMD is one whose registers leave no room beside them.  Systems in slot columns
// keep 64 per wave (their workspace has a block per 64 systems).  *sparse: at most 64
// systems per SIMD (the sparse variant's case).
template <class Prob>
int spread_lanes(int64_t n, int* lanes, bool* sparse) {
  *lanes = kLdsStride;
  *sparse = false;
  if (Prob::kColumns) return kLaunchOk;
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    return kLaunchHip;
  *lanes = systems_per_wave(n, cus, WavesPerEu<Prob>::value > 1);
  *sparse = n <= (int64_t)kLdsStride * 4 * cus;
  return kLaunchOk;
}

// Workgroups of the persistent grid: every resident slot the occupancy allows
// on every compute unit of the current device, at most one per 64 systems.
template <class Prob, int Method>
int persistent_grid(int64_t blocks, int64_t* grid) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, persistent_kernel<Prob, Method>,
                                                   kLdsStride, 0) != hipSuccess)
    return kLaunchHip;
  if (per_cu < 1) per_cu = 1;
  const int64_t g = (int64_t)cus * per_cu;
  *grid = g < blocks ? g : blocks;
  return kLaunchOk;
}

// Workspace bytes a launch needs under `schedule` (auto counts as persistent).
template <class Prob, int Method>
int64_t workspace_bytes(int schedule, int64_t n) {
  const int64_t blocks = (n + kLdsStride - 1) / kLdsStride;
  if (blocks <= 0) return 0;
  if (schedule == kSchedPlain)
    return Prob::kColumns ? (int64_t)kQueueBytes + blocks * (int64_t)block_col_bytes<Prob, Method>()
                          : 0;
  int64_t grid = 0;
  if (persistent_grid<Prob, Method>(blocks, &grid) != kLaunchOk) return -1;
  return (int64_t)kQueueBytes + grid * (int64_t)block_col_bytes<Prob, Method>();
}

template <class Prob, int Method, bool kPilot>
int launch_method(const LaunchArgs* a, hipStream_t s) {
  const int64_t blocks = (a->n + kLdsStride - 1) / kLdsStride;
  if (blocks <= 0) return kLaunchOk;
  if (blocks > 0x7fffffffLL) return kLaunchInvalid;
  const typename Prob::Params prm = a->prm;
  constexpr size_t col_bytes = block_col_bytes<Prob, Method>();
  const size_t ws_bytes = a->ws ? a->ws_bytes : 0;
  unsigned char* const ws = static_cast<unsigned char*>(a->ws);
  double* const cols = ws ? reinterpret_cast<double*>(ws + kQueueBytes) : nullptr;
  // persistent when asked, or by default when the workspace holds the queue and
  // at least one workgroup's columns
  // (the group schedule means the default one for problems without a group variant)
  const bool persistent =
      a->schedule == kSchedPersistent ||
      ((a->schedule == kSchedAuto || a->schedule == kSchedGroup) &&
       ws_bytes >= kQueueBytes + col_bytes);
  int64_t grid = 0;
  if (persistent && persistent_grid<Prob, Method>(blocks, &grid) != kLaunchOk) return kLaunchHip;
  if (persistent && ws_bytes < kQueueBytes + col_bytes) return kLaunchWorkspace;
  // a grid that holds every system at once has nothing to hand out
  if (!persistent || (!Prob::kColumns && grid == blocks)) {
    if (col_bytes && ws_bytes < kQueueBytes + (size_t)blocks * col_bytes) return kLaunchWorkspace;
    int lanes;
    bool sparse;
    if (spread_lanes<Prob>(a->n, &lanes, &sparse) != kLaunchOk) return kLaunchHip;
    const dim3 waves((unsigned)((a->n + lanes - 1) / lanes));
    if (sparse)
      plain_kernel<Sparse<Prob, Method>, Method, kPilot>
          <<<waves, dim3(kLdsStride), 0, s>>>(prm, a->n, a->y0, a->y1, a->g, a->ctl, a->status,
                                              a->stats, cols, a->order, a->carry, lanes);
    else
      plain_kernel<Prob, Method, kPilot><<<waves, dim3(kLdsStride), 0, s>>>(
          prm, a->n, a->y0, a->y1, a->g, a->ctl, a->status, a->stats, cols, a->order, a->carry,
          lanes);
    return hipGetLastError() == hipSuccess ? kLaunchOk : kLaunchHip;
  }
  if (col_bytes) {
    // a smaller workspace runs a smaller grid
    const int64_t fit = (int64_t)((ws_bytes - kQueueBytes) / col_bytes);
    if (grid > fit) grid = fit;
  }
  unsigned long long* queue = reinterpret_cast<unsigned long long*>(ws);
  queue_reset_kernel<><<<1, 1, 0, s>>>(queue);
  persistent_kernel<Prob, Method, kPilot><<<dim3((unsigned)grid), dim3(kLdsStride), 0, s>>>(
      prm, a->n, a->y0, a->y1, a->g, a->ctl, a->status, a->stats, queue, cols, a->order,
      a->carry);
  return hipGetLastError() == hipSuccess ? kLaunchOk : kLaunchHip;
}

template <class Prob>
int launch(const LaunchArgs* a, void* stream) {
  const hipStream_t s = static_cast<hipStream_t>(stream);
  if constexpr (HasGershgorin<Prob>::value && !SigmaFromGershgorin<Prob>::value) {
    if (a->method == kMethodRkc && a->ctl.sr_method == kSrGershgorin)
      return a->pilot ? launch_method<WithGershgorin<Prob>, kMethodRkc, true>(a, s)
                      : launch_method<WithGershgorin<Prob>, kMethodRkc, false>(a, s);
  }
  if (a->pilot)
    return a->method == kMethodRkck ? launch_method<Prob, kMethodRkck, true>(a, s)
                                    : launch_method<Prob, kMethodRkc, true>(a, s);
  return a->method == kMethodRkck ? launch_method<Prob, kMethodRkck, false>(a, s)
                                  : launch_method<Prob, kMethodRkc, false>(a, s);
}

template <class Prob>
int64_t workspace(int method, int schedule, int64_t n) {
  return method == kMethodRkck ? workspace_bytes<Prob, kMethodRkck>(schedule, n)
                               : workspace_bytes<Prob, kMethodRkc>(schedule, n);
}

// The per-system code of the kernels, run on the host for every system (test
// hook: the same source compiled for the CPU; each system is independent, so
// the schedule does not change any result).
template <class Prob>
int host_run(const LaunchArgs* a) {
  std::vector<double> slot((size_t)(slot_doubles<Prob, kMethodRkck>() >
                                            slot_doubles<Prob, kMethodRkc>()
                                        ? slot_doubles<Prob, kMethodRkck>()
                                        : slot_doubles<Prob, kMethodRkc>()) *
                               kLdsStride +
                           1 + SharedDoubles<Prob>::value);
  for (int k = 0; k < SharedDoubles<Prob>::value; ++k) slot[k] = crm::exp_table_entry(k);
  double* const lane = slot.data() + SharedDoubles<Prob>::value;
  for (int64_t i = 0; i < a->n; ++i) {
    if constexpr (HasGershgorin<Prob>::value && !SigmaFromGershgorin<Prob>::value) {
      if (a->method == kMethodRkc && a->ctl.sr_method == kSrGershgorin) {
        integrate_system<WithGershgorin<Prob>, kMethodRkc>(a->prm, a->n, i, a->y0, a->y1, a->g,
                                                           a->ctl, a->status, a->stats,
                                                           lane, a->carry);
        continue;
      }
    }
    if (a->method == kMethodRkck)
      integrate_system<Prob, kMethodRkck>(a->prm, a->n, i, a->y0, a->y1, a->g, a->ctl, a->status,
                                          a->stats, lane, a->carry);
    else
      integrate_system<Prob, kMethodRkc>(a->prm, a->n, i, a->y0, a->y1, a->g, a->ctl, a->status,
                                         a->stats, lane, a->carry);
  }
  return 0;
}

}  // namespace rkmi
