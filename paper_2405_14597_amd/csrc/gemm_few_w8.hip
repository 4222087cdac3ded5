// Fine-grained W8A8 GEMM, integer scales (Eq. (2) of the Integer Scale paper), up to 64 token rows: the waves of a workgroup split K.
//
// What bounds this regime: the weight stream, one byte a weight.  A workgroup takes one or two 16-row weight tiles and all of K, each of its
// waves multiplies them over its own run of K steps, the partial sums meet once in LDS.  Weights and activations are row-major, so
// both go straight to a stage of LDS that belongs to the wave alone, 8 whole 128-byte lines a load, S K steps ahead, the 16-byte chunks of a
// row permuted by (row >> 1) & 7 so that the operand reads of 16 rows fall on different banks (fetched to registers, the 16 rows
// of a tile are 16 pieces of 64 bytes a load, and every line travels twice).  A wave's loads return in order, so the waits count requests.
// The scales of a wave's run, contiguous along K in each weight row, go to LDS before everything else, a word per lane: 4 K steps
// of 16 rows a load.  One workgroup fills the compute unit's LDS, two waves a SIMD.
//
// Measured (graph replay, cold weights, N x K; the general kernel, whose operands go to registers, first): 1 row: 4096 x 14336 17.5 -> 13.8
// us (4.3 TB/s), 8192 x 28672 59.0 -> 48.9; 16 rows: 4096 x 14336 21.9 -> 15.2, 5120 x 13824 35.1 -> 19.7, 2048 x 6144 11.9 -> 6.6;
// 64 rows (every unit pulls all activations from its L2, four times the bytes of its weights): 4096 x 14336 30.3 -> 24.5, 5120 x 13824
// 53.7 -> 31.4, 8192 x 28672 83.8 -> 72.7; 0.77 of the time over 132 calls.
#include "few_common.h"
#include "tile_common.h"

namespace intscale {
namespace {

typedef int v4i_t __attribute__((ext_vector_type(4)));

constexpr int kOutOfRange = (int)0x80000000u;  // a buffer offset past every descriptor here

// Waves of a workgroup, and K steps on their way to LDS: what 160 KB hold beside the scales (64 rows and two tiles with six waves:
// 5120 x 13824 29.5 us instead of 31.4, but no room for the scales beyond K = 14336)
constexpr int waves_of(int MS, int NS) { return MS + NS > 5 ? 5 : MS + NS > 4 ? 6 : 8; }
constexpr int stages_of(int MS, int NS) { return MS + NS == 2 ? 4 : MS + NS == 3 && NS == 1 ? 3 : 2; }
constexpr size_t stage_bytes(int MS, int NS) { return (size_t)waves_of(MS, NS) * stages_of(MS, NS) * (MS + NS) * 2048; }
int scale_loads(int K, int W) { return (((K >> 7) + W - 1) / W + 3) / 4; }  // per wave and weight tile
size_t w8_lds_bytes(int K, int MS, int NS) { return stage_bytes(MS, NS) + (size_t)waves_of(MS, NS) * NS * scale_loads(K, waves_of(MS, NS)) * 256; }

// T tiles of 16 rows, one K step: 2 KB each
template <int T>
__device__ __forceinline__ void tiles_to_lds(v4i d, unsigned base, const int (&off)[2 * T], int soffset) {
    if constexpr (T >= 2) load_to_lds_rows_4x1k(d, base, off[0], off[1], off[2], off[3], soffset);
    if constexpr (T == 4) load_to_lds_rows_4x1k(d, base + 4096, off[4], off[5], off[6], off[7], soffset);
    if constexpr (T % 2 == 1) load_to_lds_rows_2x1k(d, base + (T - 1) * 2048, off[2 * T - 2], off[2 * T - 1], soffset);
}

// (two waves per SIMD: MFMA results in ordinary registers, where the scale step reads them)
template <int MS, int NS>
__global__ __launch_bounds__(waves_of(MS, NS) * kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_few_w8_kernel(FewArgs a, int quads) {
    extern __shared__ __align__(16) unsigned char smem_w8[];
    unsigned char* smem = smem_w8;
    constexpr int W = waves_of(MS, NS), S = stages_of(MS, NS), T = MS + NS, R = 2 * T;
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane & 15, kb = lane >> 4;
    const int steps = a.K >> 7, NG = a.num_groups, spg = a.group >> 7;
    const int s_begin = (wave * steps) / W, s_end = ((wave + 1) * steps) / W, count = s_end - s_begin;
    // (where the wave starts in its run differs from workgroup to workgroup: rows a power of two apart lie on one channel of the L2)
    int s_now = s_begin + ((blockIdx.x / 8) & a.phase_mask), s_ask = s_now;
    const int n0 = blockIdx.x * NS * 16, n_rows = min(NS * 16, a.N - n0);

    // ---- the scales of the wave's run: word [j][step / 4][step % 4][row]
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int scale_at = (int)stage_bytes(MS, NS) + wave * NS * quads * 256;
    const v4i sdesc = make_desc(reinterpret_cast<const int32_t*>(a.spack) + (size_t)n0 * NG, (size_t)n_rows * NG * 4);
    if (count > 0) {
        for (int q = 0; q < quads; ++q) {
            const int s = min(s_begin + 4 * q + kb, s_end - 1);
            const int g = spg == 1 ? s : s / spg;
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                const int off = (min(16 * j + li, n_rows - 1) * NG + g) * 4;
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds0 + scale_at + (j * quads + q) * 256), "v"(off), "s"(sdesc)
                             : "memory");
            }
        }
    }

    // ---- where the operands come from, and their places in a stage: token tiles, then weight tiles.  (A load's own offset of 1024 (b & 3)
    // is meant for LDS and taken off again.  Rows past the end read as zero.)
    const unsigned xbytes = (unsigned)a.M * (unsigned)a.K, wbytes = (unsigned)n_rows * (unsigned)a.K;
    const v4i xdesc = make_desc(a.xq, xbytes), wdesc = make_desc(a.wpack + (size_t)n0 * a.K, wbytes);
    int x_off[2 * MS], w_off[2 * NS];
#pragma unroll
    for (int b = 0; b < 2 * MS; ++b) {
        const int r = 8 * b + (lane >> 3);
        x_off[b] = r < a.M ? r * a.K + (((lane & 7) ^ ((r >> 1) & 7)) << 4) - (b & 3) * 1024 : kOutOfRange;
    }
#pragma unroll
    for (int b = 0; b < 2 * NS; ++b) {
        const int r = 8 * b + (lane >> 3);
        w_off[b] = r < n_rows ? r * a.K + (((lane & 7) ^ ((r >> 1) & 7)) << 4) - (b & 3) * 1024 : kOutOfRange;
    }
    const int stage_at = wave * S * T * 2048;
    int read_at[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) read_at[h] = stage_at + li * 128 + (((4 * h + kb) ^ ((li >> 1) & 7)) << 4);
    auto request = [&](int slot, int i) {
        v4i xd = xdesc, wd = wdesc;  // (past the wave's last step: nothing is fetched, zeros are written)
        xd[2] = i < count ? (int)xbytes : 0;
        wd[2] = i < count ? (int)wbytes : 0;
        const unsigned base = lds0 + stage_at + slot * T * 2048;
        tiles_to_lds<NS>(wd, base + MS * 2048, w_off, s_ask * 128);
        tiles_to_lds<MS>(xd, base, x_off, s_ask * 128);
        s_ask = s_ask + 1 == s_end ? s_begin : s_ask + 1;
    };

    v4i_t acc[MS][NS];
#pragma unroll
    for (int i = 0; i < MS; ++i)
#pragma unroll
        for (int j = 0; j < NS; ++j) acc[i][j] = v4i_t{0, 0, 0, 0};
    auto k_loop = [&](auto wide_c) {
        constexpr bool kWide = decltype(wide_c)::value;
        int slot = 0;
        for (int i_step = 0; i_step < count; ++i_step) {
            // the step's operands have come: the requests of the S - 1 steps behind it are younger
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 1) * R) : "memory");
            v4i_t xa[MS][2], wb[NS][2];
            int sc[NS];
            const int word = scale_at + ((s_now - s_begin) * 16 + li) * 4;
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                sc[j] = *reinterpret_cast<const int*>(smem + word + j * quads * 256);
#pragma unroll
                for (int h = 0; h < 2; ++h) wb[j][h] = *reinterpret_cast<const v4i_t*>(smem + read_at[h] + slot * T * 2048 + (MS + j) * 2048);
            }
#pragma unroll
            for (int i = 0; i < MS; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) xa[i][h] = *reinterpret_cast<const v4i_t*>(smem + read_at[h] + slot * T * 2048 + i * 2048);
            // (the operands are in registers: their place in LDS may be written again)
#pragma unroll
            for (int j = 0; j < NS; ++j) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(wb[j][0]), "+v"(wb[j][1]), "+v"(sc[j])::"memory");
#pragma unroll
            for (int i = 0; i < MS; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(xa[i][0]), "+v"(xa[i][1])::"memory");
            request(slot, i_step + S);
            v4i_t part[MS][NS];
#pragma unroll
            for (int j = 0; j < NS; ++j)
#pragma unroll
                for (int i = 0; i < MS; ++i) part[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][0], wb[j][0], v4i_t{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NS; ++j)
#pragma unroll
                for (int i = 0; i < MS; ++i) part[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][1], wb[j][1], part[i][j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NS; ++j)
#pragma unroll
                for (int i = 0; i < MS; ++i) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {  // C'' += C_g * s_g^INT
                        if constexpr (kWide) {
                            int prod = part[i][j][r] * sc[j];
                            asm volatile("" : "+v"(prod));  // else a 64-bit multiply-add with register pairs
                            acc[i][j][r] += prod;
                        } else {
                            acc[i][j][r] += __mul24(part[i][j][r], sc[j]);
                        }
                    }
                }
            slot = slot + 1 == S ? 0 : slot + 1;
            s_now = s_now + 1 == s_end ? s_begin : s_now + 1;
        }
    };
    if (count > 0) {
#pragma unroll
        for (int u = 0; u < S; ++u) request(u, u);
        // a scale of more than 24 signed bits among them?  (The scales are older than the S steps' requests.)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(S * R) : "memory");
        int most = 0, least = 0;
        for (int q = 0; q < NS * quads; ++q) {
            const int v = *reinterpret_cast<const int*>(smem + scale_at + q * 256 + lane * 4);
            most = max(most, v);
            least = min(least, v);
        }
        if (__any(most >= (1 << 23) || least < -(1 << 23))) k_loop(std::true_type{});
        else k_loop(std::false_type{});
    }

    // ---- the waves' partial tiles meet in LDS (nothing is on its way to the stages any more): units of one tile, in wave order
    constexpr int kUnits = MS * NS, kTurns = (kUnits + W - 1) / W;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    v4i_t* parts = reinterpret_cast<v4i_t*>(smem);
    static_assert((size_t)W * kUnits * 1024 <= stage_bytes(MS, NS), "the partial tiles take the stages' place");
    float sa[kTurns][4], c[kTurns];
    const float inv_alpha = __int_as_float((127 - a.alpha_log2) << 23);
#pragma unroll
    for (int t = 0; t < kTurns; ++t) {
        const int u = min(t * W + wave, kUnits - 1), i = u / NS, j = u - i * NS;
        c[t] = a.chan_scale ? a.chan_scale[min(n0 + 16 * j + li, a.N - 1)] : 1.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) sa[t][r] = a.a_scale[min(16 * i + 4 * kb + r, a.M - 1)];
    }
#pragma unroll
    for (int i = 0; i < MS; ++i)
#pragma unroll
        for (int j = 0; j < NS; ++j) parts[(wave * kUnits + i * NS + j) * kWave + lane] = acc[i][j];
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kTurns; ++t) {
        const int u = t * W + wave;  // (uniform over the wave)
        if (u >= kUnits) break;
        const int i = u / NS, j = u - i * NS;
        v4i_t v = parts[u * kWave + lane];
#pragma unroll
        for (int w = 1; w < W; ++w) {
            const v4i_t p = parts[(w * kUnits + u) * kWave + lane];
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] += p[r];
        }
        const int nl = 16 * j + li;
        if (nl >= n_rows) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = 16 * i + 4 * kb + r;
            if (m >= a.M) break;
            if (a.acc_out) a.acc_out[(size_t)m * a.N + n0 + nl] = v[r];
            // FLOAT(acc) * s_a[m] * c[n] / alpha (Eq. (2))
            a.out[(size_t)m * a.N + n0 + nl] = __float2half_rn((float)v[r] * sa[t][r] * (c[t] * inv_alpha));
        }
    }
}

template <int MS, int NS>
hipError_t launch_w8_instance(const FewArgs& a, hipStream_t stream) {
    static LdsLimit limit;  // per instantiation
    constexpr int W = waves_of(MS, NS);
    auto kernel = gemm_few_w8_kernel<MS, NS>;
    const hipError_t r = limit.raise(reinterpret_cast<const void*>(kernel));
    if (r != hipSuccess) return r;
    FewArgs b = a;
    b.num_groups = a.K / a.group;
    b.phase_mask = 0;  // the largest 2^n - 1 below the shortest wave's number of steps
    while (2 * b.phase_mask + 2 <= (a.K >> 7) / W) b.phase_mask = 2 * b.phase_mask + 1;
    hipLaunchKernelGGL(kernel, dim3((a.N + 16 * NS - 1) / (16 * NS)), dim3(W * kWave), w8_lds_bytes(a.K, MS, NS), stream, b, scale_loads(a.K, W));
    return hipGetLastError();
}

}  // namespace

// One weight tile a workgroup where every compute unit gets one at most, else two (1 / 2 tiles: 4096 x 14336, 16 rows, 15.2 / 19.7 us;
// 5120 x 13824 24.3 / 19.7).  K from 1024 on: with less than a step a wave, requests that fetch nothing and the longer start cost more
// (general kernel against this: 4 rows, 11080 x 256, 4.6 and 5.7 us, 17076 x 128 5.0 and 7.2).  K up to what
// leaves room in LDS for its scales (at least 32768).
int few_w8_tiles(int M, int N, int K) {
    const int ms = (M + 15) / 16, ns = (N + 15) / 16 > cu_count() ? 2 : 1;
    if (M < 1 || ms > 4 || K < 1024) return 0;
    return w8_lds_bytes(K, ms, ns) <= 160 * 1024 ? ns : 0;
}

hipError_t launch_gemm_few_w8(const FewArgs& a, hipStream_t stream) {
    const int ms = (a.M + 15) / 16, ns = few_w8_tiles(a.M, a.N, a.K);
    switch (ns == 0 ? 0 : 2 * ms + ns - 2) {
        case 1: return launch_w8_instance<1, 1>(a, stream);
        case 2: return launch_w8_instance<1, 2>(a, stream);
        case 3: return launch_w8_instance<2, 1>(a, stream);
        case 4: return launch_w8_instance<2, 2>(a, stream);
        case 5: return launch_w8_instance<3, 1>(a, stream);
        case 6: return launch_w8_instance<3, 2>(a, stream);
        case 7: return launch_w8_instance<4, 1>(a, stream);
        case 8: return launch_w8_instance<4, 2>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace intscale
