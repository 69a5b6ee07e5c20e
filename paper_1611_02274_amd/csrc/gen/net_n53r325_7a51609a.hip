// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Launchers of the 53-species network (topology n53r325_7a51609a).
#include "net_n53r325_7a51609a.hpp"

extern "C" int rkmi_gen_n53r325_7a51609a_launch(const rkmi::LaunchArgs* a, void* s) {
  return rkmi::launch_with_wide<rkmi::gen_n53r325_7a51609a::Net, rkmi::gen_n53r325_7a51609a::GNet, rkmi::gen_n53r325_7a51609a::WNet>(a, s);
}

extern "C" int rkmi_gen_n53r325_7a51609a_host(const rkmi::LaunchArgs* a) {
  return rkmi::host_run<rkmi::gen_n53r325_7a51609a::Net>(a);
}

extern "C" int64_t rkmi_gen_n53r325_7a51609a_workspace(int method, int schedule, int64_t n) {
  return rkmi::workspace_with_group<rkmi::gen_n53r325_7a51609a::Net, rkmi::gen_n53r325_7a51609a::GNet>(method, schedule, n);
}
