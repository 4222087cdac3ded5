// Interface of the kernels for few token rows whose waves split K (gemm_few_pk.hip; int8 weights: gemm_few_w8.hip).
#pragma once
#include "is_common.h"

namespace intscale {

struct FewArgs {
    const int8_t* xq;         // [M,K]
    const float* a_scale;     // [M]
    const uint8_t* wpack;     // kernel layout
    const uint8_t* spack;     // kernel layout (header included)
    const float* chan_scale;  // [N] or nullptr
    __half* out;              // [M,N], or [M,N/2] with the SiLU * up epilogue
    int32_t* acc_out;         // [M,N] or nullptr
    int M, N, K, group;
    int alpha_log2;
    int num_groups = 0, phase_mask = 0;  // set by the launcher
};

struct FewPlan {
    int ms;     // 16-row token tiles
    int ns;     // 16-row weight tiles of a workgroup
    int waves;  // waves of a workgroup (the K split)
    int depth;  // K steps whose weights a wave has on their way
    double us = 0.0;  // few_plan: fitted time of its loops and ends
};

// Mixture-of-experts form: xq / a_scale / out hold all experts' rows sorted by expert, expert e owning rows
// [row_offsets[e], row_offsets[e+1]); wpack, spack and chan_scale of FewArgs are expert 0's.
struct FewGroups {
    const int32_t* row_offsets;  // device, [num_experts + 1]
    int num_experts;
    size_t wstride, sstride;     // bytes from one expert's packed weights / scales to the next
};

FewPlan few_plan(int M, int N, int K, bool silu);
void few_kernel_name(const FewPlan& p, bool int_scale, bool silu, char* buf, size_t len);
hipError_t launch_gemm_few_pk(const FewArgs& a, const FewPlan& p, bool int_scale, bool silu, hipStream_t stream);
// The same on several tiles of 48 or 64 rows (65 rows and more, integer scales)
FewPlan rows_plan(int M, int N, int K, bool silu, double* us_out);
void rows_kernel_name(const FewPlan& p, bool silu, char* buf, size_t len);
hipError_t launch_gemm_rows_pk(const FewArgs& a, const FewPlan& p, bool silu, hipStream_t stream);
// (ms: 16-row token tiles a workgroup takes at a time; ns = 0: the call is not for this kernel)
FewPlan few_grouped_plan(int E, int M, int N, int K);
void few_grouped_kernel_name(const FewPlan& p, bool int_scale, char* buf, size_t len);
hipError_t launch_gemm_few_grouped_pk(const FewArgs& a, const FewGroups& g, const FewPlan& p, bool int_scale, hipStream_t stream);
// Row-major int8 weights in `wpack`, row-major integer scales in `spack` (gemm_few_w8.hip): weight tiles of a workgroup, 0 where the call
// is not for this kernel
int few_w8_tiles(int M, int N, int K);
hipError_t launch_gemm_few_w8(const FewArgs& a, hipStream_t stream);

}  // namespace intscale
