// Interface of the kernel whose waves split K (gemm_wavek.hip): int4 weights in the kernel layout, or int8 weights in the
// canonical one, on quantised activations.
#pragma once
#include "is_common.h"

namespace intscale {

struct WavekArgs {
    const int8_t* xp;         // quantised activations in the blocks of the preparation kernels [16-row tile][K step], 2 KB each
    const float* a_scale;     // [M]
    const void* w;            // kernel layout (int4), or codes [N,K] (int8)
    const void* scale;        // kernel layout without its header, or [N,NG]
    const void* flags;        // the kernel layout's header (int4 with integer scales)
    const float* chan_scale;  // [N] or nullptr
    __half* out;              // [M,N], or [M,N/2] with the SiLU * up epilogue
    int32_t* acc_out;         // [M,N] or nullptr
    int M, N, K, group;
    int alpha_log2;
};

struct WavekPlan {
    int ms;                  // 16-row token sub-tiles of a tile
    int waves;               // waves of a workgroup (the K split)
    long long tiles;         // workgroups
    double us;               // its fitted time
    bool by_padding = true;  // the row tiles that pad least
};

bool takes_wavek(int M, int N, int K, bool w8 = false);  // the dispatch of the tiled kernel's calls (api.hip)
bool wavek_is_faster(int M, int N, int K, bool w8);
double prepared_gemm_us(int M, int N, int K);  // a GEMM call of more than 64 rows on prepared activations, with their preparation
WavekPlan wavek_plan(int M, int N, int K, bool w8);
void wavek_kernel_name(const WavekPlan& p, bool int_scale, bool w8, bool silu, char* buf, size_t len);
hipError_t launch_gemm_wavek(const WavekArgs& a, const WavekPlan& p, bool int_scale, bool w8, bool silu, hipStream_t stream);

}  // namespace intscale
