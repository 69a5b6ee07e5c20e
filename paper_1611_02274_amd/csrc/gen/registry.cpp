// Generated by paper_1611_02274_amd/codegen.py -- do not edit.
// Networks compiled into the library, matched by exact topology.
#include "../rk_types.hpp"

extern "C" int rkmi_gen_n9r19_49a69f7b_th_launch(const rkmi::LaunchArgs*, void*);
extern "C" int rkmi_gen_n9r19_49a69f7b_th_host(const rkmi::LaunchArgs*);
extern "C" int64_t rkmi_gen_n9r19_49a69f7b_th_workspace(int, int, int64_t);
extern "C" int rkmi_gen_n13r27_7b5c2807_th_launch(const rkmi::LaunchArgs*, void*);
extern "C" int rkmi_gen_n13r27_7b5c2807_th_host(const rkmi::LaunchArgs*);
extern "C" int64_t rkmi_gen_n13r27_7b5c2807_th_workspace(int, int, int64_t);
extern "C" int rkmi_gen_n32r133_bcb31e07_th_launch(const rkmi::LaunchArgs*, void*);
extern "C" int rkmi_gen_n32r133_bcb31e07_th_host(const rkmi::LaunchArgs*);
extern "C" int64_t rkmi_gen_n32r133_bcb31e07_th_workspace(int, int, int64_t);
namespace rkmi { RateOrder gen_n32r133_bcb31e07_th_rates(int); }
extern "C" int rkmi_gen_n53r325_7a51609a_th_launch(const rkmi::LaunchArgs*, void*);
extern "C" int rkmi_gen_n53r325_7a51609a_th_host(const rkmi::LaunchArgs*);
extern "C" int64_t rkmi_gen_n53r325_7a51609a_th_workspace(int, int, int64_t);
namespace rkmi { RateOrder gen_n53r325_7a51609a_th_rates(int); }
extern "C" int rkmi_gen_n9r19_49a69f7b_launch(const rkmi::LaunchArgs*, void*);
extern "C" int rkmi_gen_n9r19_49a69f7b_host(const rkmi::LaunchArgs*);
extern "C" int64_t rkmi_gen_n9r19_49a69f7b_workspace(int, int, int64_t);
extern "C" int rkmi_gen_n9r19_49a69f7b_taped(const rkmi::LaunchArgs*, const rkmi::TapeArgs*, void*);
extern "C" int rkmi_gen_n9r19_49a69f7b_taped_host(const rkmi::LaunchArgs*, const rkmi::TapeArgs*);
extern "C" int rkmi_gen_n9r19_49a69f7b_adjoint(const rkmi::AdjointArgs*, void*);
extern "C" int rkmi_gen_n9r19_49a69f7b_adjoint_host(const rkmi::AdjointArgs*);
extern "C" int rkmi_gen_n13r27_7b5c2807_launch(const rkmi::LaunchArgs*, void*);
extern "C" int rkmi_gen_n13r27_7b5c2807_host(const rkmi::LaunchArgs*);
extern "C" int64_t rkmi_gen_n13r27_7b5c2807_workspace(int, int, int64_t);
extern "C" int rkmi_gen_n13r27_7b5c2807_taped(const rkmi::LaunchArgs*, const rkmi::TapeArgs*, void*);
extern "C" int rkmi_gen_n13r27_7b5c2807_taped_host(const rkmi::LaunchArgs*, const rkmi::TapeArgs*);
extern "C" int rkmi_gen_n13r27_7b5c2807_adjoint(const rkmi::AdjointArgs*, void*);
extern "C" int rkmi_gen_n13r27_7b5c2807_adjoint_host(const rkmi::AdjointArgs*);
extern "C" int rkmi_gen_n32r133_bcb31e07_launch(const rkmi::LaunchArgs*, void*);
extern "C" int rkmi_gen_n32r133_bcb31e07_host(const rkmi::LaunchArgs*);
extern "C" int64_t rkmi_gen_n32r133_bcb31e07_workspace(int, int, int64_t);
extern "C" int rkmi_gen_n53r325_7a51609a_launch(const rkmi::LaunchArgs*, void*);
extern "C" int rkmi_gen_n53r325_7a51609a_host(const rkmi::LaunchArgs*);
extern "C" int64_t rkmi_gen_n53r325_7a51609a_workspace(int, int, int64_t);
extern "C" int rkmi_batch_61d6bd15_launch(const rkmi::BatchArgs*, void*);
extern "C" int64_t rkmi_batch_61d6bd15_workspace(const rkmi::BatchArgs*);
extern "C" void rkmi_batch_61d6bd15_free(void*);

static const int32_t reac_n9r19_49a69f7b[] = {3, 8, 1, 7, 6, -1, 7, -1, 0, 5, 4, -1, 3, 7, 8, -1, 2, 4, 2, 8, 0, 2, 2, 6, 3, 7, 8, -1, 2, 3, 1, 8, 3, 4, 0, 7, 5, 8};
static const int32_t prod_n9r19_49a69f7b[] = {6, 6, 4, 5, 0, 5, 2, 6, 3, 3, 1, 3, 5, 6, 3, 6, 1, 5, 5, 6, 3, -1, 3, 5, 2, 8, 0, 7, 5, -1, 4, 6, 1, 6, 3, 6, 6, 7};
static const int32_t reac_n13r27_7b5c2807[] = {3, 5, 0, 5, 3, 8, 1, 5, 0, 9, 4, 8, 9, -1, 6, 6, 6, -1, 2, 3, 0, 5, 0, 8, 7, 12, 0, 2, 9, -1, 4, 8, 6, 8, 0, 7, 4, -1, 0, 9, 10, 10, 4, 5, 0, 10, 1, 8, 8, 8, 2, 9, 5, 6};
static const int32_t prod_n13r27_7b5c2807[] = {0, 6, 3, 8, 6, -1, 8, 10, 6, 8, 3, 5, 5, 8, 4, 9, 2, 4, 5, -1, 2, 4, 5, -1, 2, 11, 8, -1, 2, 6, 0, 6, 5, 5, 1, 10, 0, 3, 5, 5, 3, 7, 3, 6, 1, 3, 2, 10, 2, 5, 12, -1, 3, 9};
static const int32_t reac_n32r133_bcb31e07[] = {8, 15, 15, 30, 12, 28, 22, 23, 9, 25, 6, 21, 10, 21, 3, 26, 26, 28, 8, 21, 11, 14, 9, 16, 9, 24, 11, 17, 1, 22, 16, 21, 7, 20, 2, 2, 27, -1, 16, 21, 24, 31, 20, 21, 9, 29, 10, 28, 4, 17, 22, -1, 24, 27, 0, 26, 1, 9, 9, 15, 20, 26, 23, 31, 10, 21, 14, 25, 6, 18, 2, 26, 3, 22, 16, 26, 1, 26, 5, 13, 2, 28, 13, 28, 26, 27, 16, 24, 10, 31, 4, 30, 18, 19, 3, 7, 10, 21, 4, 16, 19, 22, 1, 27, 5, 14, 14, 23, 20, 27, 22, 30, 3, 27, 5, 12, 3, 26, 15, 22, 20, 31, 15, 20, 23, 30, 25, 25, 15, 21, 28, 31, 2, 25, 7, 11, 9, 29, 4, 7, 3, 26, 14, 23, 3, 31, 8, 26, 1, 21, 4, 30, 7, 22, 16, -1, 12, 30, 8, -1, 14, 30, 4, 4, 9, 20, 6, 17, 5, 16, 12, 14, 14, 30, 16, 17, 28, -1, 2, 10, 31, -1, 5, 25, 20, 20, 16, 24, 17, 23, 9, 24, 2, 9, 3, 16, 2, 5, 2, 20, 14, 19, 8, 29, 5, 10, 3, 15, 11, 25, 14, 21, 3, 4, 14, 30, 17, 24, 16, 30, 11, 13, 1, 16, 15, 20, 4, 16, 30, -1, 11, 31, 12, -1, 21, 27, 1, 26, 1, 17, 0, 27, 4, 26, 12, 14, 22, 25, 4, 26, 17, 20, 10, 17, 25, 28, 7, 28, 3, 9, 16, 22, 10, 28, 22, 31};
static const int32_t prod_n32r133_bcb31e07[] = {4, 23, 6, 7, 17, 17, 4, 27, 23, 27, 14, 19, 3, 26, 13, 28, 21, 25, 5, 9, 2, 24, 7, 25, 18, 28, 5, 13, 2, 21, 14, 25, 10, 28, 11, -1, 6, 21, 17, 20, 20, 22, 3, 17, 18, 20, 14, 19, 5, 7, 3, 14, 12, 14, 2, 9, 15, 25, 19, 28, 8, 13, 19, 28, 15, 18, 23, 24, 7, 13, 13, 31, 14, 14, 6, 12, 16, 16, 10, 22, 14, 15, 19, 24, 12, 25, 10, 22, 16, 20, 1, 17, 6, 12, 2, 8, 14, 30, 20, 31, 14, 25, 6, 17, 4, 22, 8, 20, 21, 30, 18, 31, 17, 20, 22, 27, 12, -1, 5, 20, 3, 7, 4, 6, 19, 25, 9, 30, 3, 8, 4, 8, 26, -1, 4, 13, 13, 21, 20, 28, 9, 11, 15, 17, 2, 28, 17, 25, 4, 16, 3, 25, 14, 17, 0, 10, 26, 26, 0, 7, 13, 28, 0, 5, 8, 16, 30, 31, 20, 21, 18, 21, 12, -1, 12, 15, 4, 15, 6, 11, 0, 20, 9, 14, 6, 14, 3, 18, 8, 25, 4, 12, 1, 17, 20, 20, 0, 24, 11, 15, 2, 9, 3, 18, 6, 22, 1, 4, 2, 26, 24, 28, 0, 14, 2, 27, 5, 18, 10, 25, 10, 29, 6, 20, 1, 31, 17, -1, 1, 16, 1, 24, 19, 24, 12, 28, 7, 10, 7, 20, 5, 19, 19, 22, 22, 26, 14, 27, 5, 30, 19, 22, 20, 26, 9, 31, 8, 31, 5, 19, 7, 24, 3, 25, 24, 28};
static const int32_t reac_n53r325_7a51609a[] = {16, 48, 13, 26, 9, 45, 17, 34, 5, 37, 1, 38, 9, 32, 14, 40, 18, -1, 16, 24, 24, 31, 8, 35, 10, 39, 33, 52, 13, 13, 28, 46, 7, 42, 14, 14, 14, 17, 8, 30, 37, 52, 11, 12, 4, 47, 14, 36, 24, 33, 2, 25, 0, 43, 3, 32, 13, 23, 9, 35, 26, 33, 5, 41, 13, 45, 9, 39, 8, 13, 4, 31, 28, 39, 20, 23, 8, 35, 14, 17, 14, 33, 16, 20, 13, 33, 20, 29, 27, 46, 3, 41, 27, 49, 6, 46, 3, 50, 16, 36, 16, 38, 40, 46, 20, 23, 17, 33, 49, 50, 6, 31, 23, 23, 11, 23, 0, 52, 22, 39, 17, 33, 6, 45, 4, 45, 0, 26, 1, 18, 2, 19, 11, 23, 2, 43, 7, 52, 18, 19, 4, 9, 40, 48, 28, 33, 4, 21, 17, 40, 13, 45, 22, 47, 7, 16, 11, 39, 48, 50, 43, -1, 10, 50, 17, 34, 9, 12, 2, 35, 24, 46, 25, 35, 9, 26, 7, 18, 33, 50, 2, 43, 22, 51, 43, -1, 36, 52, 1, 18, 22, 37, 35, 52, 27, 28, 3, 32, 4, 27, 7, 18, 18, 19, 27, 40, 24, 28, 1, 1, 4, 49, 23, 41, 16, 32, 1, 20, 6, 45, 9, 48, 13, 48, 12, 38, 1, 9, 28, 38, 38, 45, 15, 23, 20, 34, 20, 23, 1, 32, 14, 25, 23, 33, 42, -1, 38, -1, 13, 33, 35, 42, 2, 21, 29, 37, 12, 12, 19, 31, 7, 41, 11, 44, 2, 26, 33, 40, 12, 43, 9, 16, 42, 52, 11, 23, 5, 48, 24, 48, 38, 42, 30, 45, 43, -1, 21, 51, 43, 51, 26, 46, 13, 31, 3, 13, 26, 28, 4, 10, 8, 26, 9, 49, 28, 51, 16, 38, 7, 24, 15, 47, 14, 52, 8, 9, 34, 46, 3, 20, 20, 45, 5, 52, 30, -1, 15, 17, 8, 47, 12, 26, 9, 49, 8, 42, 39, 40, 33, 41, 9, 39, 20, 27, 28, 32, 12, 20, 14, 31, 24, 27, 16, 51, 27, 36, 11, 48, 1, 24, 23, 49, 22, 37, 13, 33, 0, 29, 36, 36, 3, 7, 22, 47, 9, 14, 9, 38, 20, 38, 9, 11, 6, 38, 6, 37, 17, 22, 28, 51, 1, 42, 1, 21, 8, 44, 2, 43, 14, 38, 7, 15, 11, 48, 22, 51, 48, 50, 11, 25, 32, 46, 19, 33, 4, 35, 12, 37, 10, 47, 12, 41, 19, 22, 14, 22, 25, 26, 24, 36, 12, 46, 12, 15, 13, 49, 1, 5, 13, 52, 4, 27, 19, 19, 0, 16, 30, 37, 9, 49, 20, 33, 14, 18, 14, 27, 14, 19, 24, 42, 7, 27, 31, -1, 27, 42, 20, 52, 27, 33, 1, 35, 14, 30, 6, 16, 40, 51, 4, 22, 12, 43, 18, 39, 10, 31, 19, 32, 23, 25, 15, 51, 4, 23, 10, 51, 5, 48, 11, 33, 10, 39, 19, 45, 10, 30, 19, 35, 12, 43, 8, 43, 20, 23, 17, 36, 11, 21, 15, 17, 29, 31, 12, 25, 21, 45, 24, 25, 22, 52, 12, 14, 23, 24, 26, 50, 18, 50, 19, 23, 9, 45, 17, 18, 19, 41, 13, 25, 40, 43, 29, 37, 2, 46, 1, 11, 27, 44, 18, 29, 9, 17, 19, 20, 33, 35, 40, 48, 8, 29, 7, 32, 17, 27, 19, 49, 1, 11, 27, 36, 36, 52, 17, 21, 22, 48, 11, 27, 33, 33, 8, 12, 29, 33, 23, 52, 0, 22, 34, 43, 15, 47, 25, 50, 35, 43, 8, 19, 34, 38, 5, 24, 1, 4, 23, 38, 37, 52, 35, 46, 31, 42, 25, 36, 29, 32, 14, 37, 2, 22, 15, 46, 15, 38, 16, 30, 25, 43, 8, 51, 11, 27, 18, 45, 22, -1, 2, 5, 28, 52};
static const int32_t prod_n53r325_7a51609a[] = {7, 31, 16, 31, 19, 33, 5, 51, 19, 28, 7, 25, 22, 44, 11, 27, 7, 14, 11, 31, 39, 43, 16, 16, 32, 50, 31, 47, 7, 35, 8, 37, 9, 28, 19, 40, 9, 47, 6, 32, 25, 33, 5, 19, 5, 51, 18, 25, 21, 23, 23, -1, 13, 16, 12, 43, 34, 44, 37, 40, 23, 32, 30, 42, 37, 52, 10, 52, 0, 15, 12, 43, 42, 45, 36, 50, 5, 36, 12, 13, 31, 50, 10, 13, 16, 48, 18, 19, 16, 51, 8, 30, 31, 47, 2, 16, 0, 6, 18, 33, 8, 36, 9, 23, 0, 21, 12, 44, 27, 37, 14, 29, 34, 49, 14, 22, 1, 23, 15, 52, 7, 45, 40, 47, 9, 52, 4, 49, 20, 27, 12, 50, 18, 34, 14, 16, 16, 51, 21, 50, 3, 10, 9, 39, 8, 36, 15, 19, 3, 33, 19, 49, 3, 31, 14, 20, 15, 27, 7, 25, 8, 25, 7, 8, 4, 47, 0, 14, 4, 25, 8, 49, 16, 45, 15, 25, 8, 37, 2, 36, 34, 38, 17, 29, 3, 36, 33, 39, 9, 25, 10, 35, 27, 31, 24, 50, 18, 27, 12, 40, 28, 46, 5, 44, 23, 34, 11, 21, 51, -1, 14, 33, 24, 31, 13, 41, 0, 46, 25, 34, 20, 25, 33, 46, 13, 19, 2, 46, 37, 42, 33, 33, 8, 26, 9, 14, 13, 13, 36, 47, 3, 49, 29, 48, 2, 28, 1, 10, 9, 49, 24, 28, 3, 36, 19, 21, 2, 47, 25, 35, 13, 21, 7, 43, 14, 23, 13, 29, 13, 29, 8, 13, 22, 23, 8, 29, 1, 15, 21, 25, 18, 28, 31, 52, 2, 21, 19, 49, 29, 48, 30, 37, 19, 32, 14, 50, 8, 41, 5, 20, 14, 43, 16, 48, 3, 44, 42, 48, 11, 48, 2, 41, 12, 30, 28, 50, 14, 19, 9, 50, 25, 37, 23, 34, 50, 52, 0, 43, 2, 35, 14, 39, 14, 44, 11, 28, 31, 34, 21, 31, 18, 47, 14, 46, 18, 21, 7, 19, 24, 25, 39, 40, 12, 33, 25, 35, 5, 44, 19, 23, 33, 39, 13, 18, 10, 45, 12, 16, 21, 44, 0, 4, 14, 23, 1, 42, 16, 20, 10, 37, 8, 8, 10, 34, 0, 22, 16, 19, 14, 46, 16, 50, 20, 52, 20, 35, 5, 33, 5, 44, 11, 37, 37, 40, 3, 49, 0, 33, 5, 33, 31, 37, 12, 36, 5, 33, 48, 50, 0, 35, 16, 39, 8, 23, 16, 40, 24, 45, 13, 41, 33, -1, 24, 50, 31, 46, 3, 19, 24, 51, 5, 47, 1, 16, 2, 38, 33, 35, 0, 32, 13, 37, 13, 22, 3, 39, 11, 51, 11, 43, 9, 47, 45, 50, 4, 24, 23, 46, 19, 39, 31, -1, 22, 52, 8, 34, 1, 29, 28, 34, 15, 47, 30, 38, 15, 48, 33, 35, 13, 52, 41, -1, 3, 35, 48, 50, 4, 33, 16, 16, 13, 35, 1, 31, 18, 23, 27, 38, 19, 24, 24, 28, 7, 35, 19, 44, 8, 43, 25, 28, 43, 52, 1, 23, 36, 39, 13, 30, 31, 34, 27, 50, 15, 52, 22, 25, 4, 38, 0, 30, 18, 51, 10, 25, 16, 31, 20, 52, 22, 24, 32, 50, 13, -1, 0, 40, 37, 52, 39, 42, 0, 13, 10, 17, 38, 39, 1, 43, 14, 22, 35, 37, 0, 52, 37, 52, 22, -1, 23, 33, 35, 45, 20, 39, 24, 46, 6, 35, 25, 36, 22, -1, 13, 30, 30, 47, 11, 17, 11, 30, 18, 27, 9, 47, 18, 26, 2, 18, 3, 21, 22, 40, 3, 17, 8, 49, 21, 51, 20, 39, 8, 41, 38, 45, 24, 31, 36, 50, 3, 16, 13, 18, 36, 42, 31, 40, 24, 33, 25, 50, 3, 24, 26, 46, 0, 40, 6, 50, 5, 49};

namespace rkmi {
extern const GenEntry kGenRegistry[] = {
    {9, 19, reac_n9r19_49a69f7b, prod_n9r19_49a69f7b, rkmi_gen_n9r19_49a69f7b_launch, rkmi_gen_n9r19_49a69f7b_host, rkmi_gen_n9r19_49a69f7b_workspace, rkmi_gen_n9r19_49a69f7b_taped, rkmi_gen_n9r19_49a69f7b_taped_host, rkmi_gen_n9r19_49a69f7b_adjoint, rkmi_gen_n9r19_49a69f7b_adjoint_host, 0, nullptr},
    {13, 27, reac_n13r27_7b5c2807, prod_n13r27_7b5c2807, rkmi_gen_n13r27_7b5c2807_launch, rkmi_gen_n13r27_7b5c2807_host, rkmi_gen_n13r27_7b5c2807_workspace, rkmi_gen_n13r27_7b5c2807_taped, rkmi_gen_n13r27_7b5c2807_taped_host, rkmi_gen_n13r27_7b5c2807_adjoint, rkmi_gen_n13r27_7b5c2807_adjoint_host, 0, nullptr},
    {32, 133, reac_n32r133_bcb31e07, prod_n32r133_bcb31e07, rkmi_gen_n32r133_bcb31e07_launch, rkmi_gen_n32r133_bcb31e07_host, rkmi_gen_n32r133_bcb31e07_workspace, nullptr, nullptr, nullptr, nullptr, 0, nullptr},
    {53, 325, reac_n53r325_7a51609a, prod_n53r325_7a51609a, rkmi_gen_n53r325_7a51609a_launch, rkmi_gen_n53r325_7a51609a_host, rkmi_gen_n53r325_7a51609a_workspace, nullptr, nullptr, nullptr, nullptr, 0, nullptr},
    {9, 19, reac_n9r19_49a69f7b, prod_n9r19_49a69f7b, rkmi_gen_n9r19_49a69f7b_th_launch, rkmi_gen_n9r19_49a69f7b_th_host, rkmi_gen_n9r19_49a69f7b_th_workspace, nullptr, nullptr, nullptr, nullptr, 1, nullptr},
    {13, 27, reac_n13r27_7b5c2807, prod_n13r27_7b5c2807, rkmi_gen_n13r27_7b5c2807_th_launch, rkmi_gen_n13r27_7b5c2807_th_host, rkmi_gen_n13r27_7b5c2807_th_workspace, nullptr, nullptr, nullptr, nullptr, 1, nullptr},
    {32, 133, reac_n32r133_bcb31e07, prod_n32r133_bcb31e07, rkmi_gen_n32r133_bcb31e07_th_launch, rkmi_gen_n32r133_bcb31e07_th_host, rkmi_gen_n32r133_bcb31e07_th_workspace, nullptr, nullptr, nullptr, nullptr, 1, gen_n32r133_bcb31e07_th_rates},
    {53, 325, reac_n53r325_7a51609a, prod_n53r325_7a51609a, rkmi_gen_n53r325_7a51609a_th_launch, rkmi_gen_n53r325_7a51609a_th_host, rkmi_gen_n53r325_7a51609a_th_workspace, nullptr, nullptr, nullptr, nullptr, 1, gen_n53r325_7a51609a_th_rates},
};
extern const int kGenRegistrySize = 8;
extern const BatchEntry kBatchRegistry[] = {
    {4, {0, 1, 2, 3}, rkmi_batch_61d6bd15_launch, rkmi_batch_61d6bd15_workspace, rkmi_batch_61d6bd15_free},
};
extern const int kBatchRegistrySize = 1;
}  // namespace rkmi
