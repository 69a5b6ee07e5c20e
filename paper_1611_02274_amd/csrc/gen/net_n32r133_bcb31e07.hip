// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Launchers of the 32-species network (topology n32r133_bcb31e07).
#include "net_n32r133_bcb31e07.hpp"

extern "C" int rkmi_gen_n32r133_bcb31e07_launch(const rkmi::LaunchArgs* a, void* s) {
  return rkmi::launch_with_wide<rkmi::gen_n32r133_bcb31e07::Net, rkmi::gen_n32r133_bcb31e07::GNet, rkmi::gen_n32r133_bcb31e07::WNet>(a, s);
}

extern "C" int rkmi_gen_n32r133_bcb31e07_host(const rkmi::LaunchArgs* a) {
  return rkmi::host_run<rkmi::gen_n32r133_bcb31e07::Net>(a);
}

extern "C" int64_t rkmi_gen_n32r133_bcb31e07_workspace(int method, int schedule, int64_t n) {
  return rkmi::workspace_with_group<rkmi::gen_n32r133_bcb31e07::Net, rkmi::gen_n32r133_bcb31e07::GNet>(method, schedule, n);
}
