// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Launchers of the 32-species network with the energy equation (topology n32r133_bcb31e07_th): the
// group kernels under every schedule; no host build of the per-system code.
#include "net_n32r133_bcb31e07_th.hpp"

extern "C" int rkmi_gen_n32r133_bcb31e07_th_launch(const rkmi::LaunchArgs* a, void* s) {
  return rkmi::launch_group_only<rkmi::gen_n32r133_bcb31e07_th::GNet, rkmi::gen_n32r133_bcb31e07_th::WNet>(a, s);
}

extern "C" int rkmi_gen_n32r133_bcb31e07_th_host(const rkmi::LaunchArgs*) {
  return rkmi::kLaunchInvalid;
}

extern "C" int64_t rkmi_gen_n32r133_bcb31e07_th_workspace(int, int, int64_t n) {
  return n > 0 ? (int64_t)rkmi::kQueueBytes : 0;
}

namespace rkmi {
RateOrder gen_n32r133_bcb31e07_th_rates(int k) {
  using G = gen_n32r133_bcb31e07_th::GNet;
  using W = gen_n32r133_bcb31e07_th::WNet;
  return k == 0 ? RateOrder{G::kRxOf, G::R * G::kL, G::kPrmOffset}
                : RateOrder{W::kRxOf, W::R * W::kL, W::kPrmOffset};
}
}  // namespace rkmi
