// Fine-grained W4A8 and W8A8 GEMM for a moderate number of token rows (a prompt's chunk, a large decode batch): the
// waves of a workgroup split K.  Integer-scale form: Eq. (2) / Table 2 "Ours" of the Integer Scale paper; float-scale form:
// Eq. (1) / Table 2 "Atom".
//
// What bounds this regime.  A few hundred token rows make a few dozen tiles of 128 x 256, far fewer than the chip has
// compute units; cutting their K range over workgroups moves partial tiles of 128 KB through memory, and one workgroup per tile
// adds them up while the others are done (300 x 4096 x 4096: 8 K steps a workgroup, 31 us).  Here a workgroup owns a
// small output tile (up to 80 x 64) over all of K, each of its waves multiplies the whole tile over its own run of K steps,
// and the partial tiles meet in LDS.  300 rows make 320 workgroups of 4096 columns, no partial tile leaves the compute
// unit, and no wave waits for another before the end: there is no barrier in the K loop.
//
// Operands go straight from global memory to the registers of the wave that multiplies them (no two waves of a workgroup
// read the same bytes, so LDS would only pass them on): weights in the 1 KB blocks of the kernel layout, activations in the
// 2 KB blocks that the preparation kernels write, every load one contiguous kilobyte.  (Row-major activations, which
// need no preparation, cost 71 cycles per load and compute unit in 16 pieces of 64 bytes against about 30: 2048 x 28672 x 4096
// 519 against 344 us, and no gain at 65 rows.)  Each register is asked for again as soon as its last use has been
// issued, a K step ahead; two waves per SIMD cover the rest of the latency.  What bounds it, from counters: with int4 weights
// (300 x 28672 x 4096, 58 us) a wave issues 43 % of its time, waits for an issue slot 37 % and for loads 21 %, so that the two
// waves of a SIMD leave it little room, and the L2 delivers 34 bytes per cycle and compute unit (14 KB of operands per 40 MFMAs
// of a wave; tile loads alone sustain 40 to 55): large calls stay on the tiled kernel, which shares its operands through LDS
// (takes_wavek says where the line lies).  With int8 weights (300 x 4096 x 14336, 42 us) it waits for loads: 48 % of a wave's
// time, 34 % issuing, 28 bytes per cycle.  There the weight lines are requested by assembly, which the compiler does not
// count, so that its waits for the activations (7 and 6 outstanding) hold up until the lines just requested have come too: they
// are less than a K step ahead; and the copy of the scales every fourth step waits for everything.
//
// int4 -> int8 with a zero point, as in the tiled kernel: (word ^ 0x08..) & 0x0F.. is q + 8, and the MFMA chain starts from
// -8 * sum_k x[m,k].  That sum comes from the matrix pipe as well (a multiplication by a constant operand of -8s gives it in every
// column): 2 MFMAs per 8, where loading the preparation's sums costs a request per sub-tile (M = 300, 4096 x 14336:
// 43.7 with the loads, 41.7 us without).
//
// Measured (GEMM on int8 codes, its preparation included, graph replay), the tiled kernel's time first: 65 x 4096 x 4096
// 32.9 -> 12.6 us, 300 x 4096 x 4096 36.4 -> 19.5 us, 512 x 6144 x 4096 42.2 -> 28.5 us, 300 x 28672 x 4096 72.9 -> 58.2 us,
// 128 x 4096 x 14336 46.2 -> 25.0 us, 300 x 4096 x 14336 32.4 us (41.9 in tiles of 64 rows); W8A8 300 x 4096 x 14336 122 -> 42 us,
// 1024 x 4096 x 14336 128 -> 108 us; W4A8 1024 x 28672 x 4096 147 against 181 us (stays on the tiled kernel).
#include <math.h>
#include <stdio.h>

#include <algorithm>

#include "act_common.h"
#include "pk_common.h"
#include "tile_common.h"
#include "wavek_common.h"

namespace intscale {
namespace {

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef float v4f_t __attribute__((ext_vector_type(4)));

constexpr int kNS = 4;                // 16-row weight sub-tiles of a tile: 64 output columns
constexpr int kTN = kNS * 16;
constexpr int kPitch = kTN + 8;       // halves per row of the output tile in LDS

constexpr int kStage8 = kTN * 128;    // int8 weights of one K step
// Token sub-tiles whose partial sums pass through LDS at a time: all of them up to 64 rows; all five of 80 would need 160 KB with
// eight waves, and with four leave no room for the second workgroup on the unit
constexpr int rows_at_once(int MS, int W) { return W * MS * kNS > 16 * W ? (MS + 1) / 2 : MS; }
constexpr size_t sums_bytes(int MS, int W) { return (size_t)W * rows_at_once(MS, W) * kNS * 1024; }
constexpr size_t lds_bytes(int MS, int W, bool W8) {
    const size_t sums = sums_bytes(MS, W) + (size_t)MS * 16 * kPitch * 2, stages = W8 ? (size_t)W * 2 * kStage8 : 0;
    return sums > stages ? sums : stages;
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes > 0x7FFFFFFFull ? 0x7FFFFFFFu : (unsigned)bytes,
                                             0x00020000);
}

// MS: 16-row token sub-tiles of a tile.  W: waves.  W8: int8 weights and scales in their canonical layouts.  WIDE: 32-bit
// multiplies in the integer scale step (some scale does not fit 24 signed bits).
template <bool INT_SCALE, bool WIDE, bool W8, int MS, int W, bool SILU>
__device__ __forceinline__ void wavek_tile(const WavekArgs& a, unsigned char* smem) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane & 15, kb = lane >> 4;
    const int tiles_n = (a.N + kTN - 1) / kTN, tiles_m = (a.M + MS * 16 - 1) / (MS * 16);
    const TileAt tile = tile_of_block(blockIdx.x, tiles_m, tiles_n);
    const int m0 = tile.m * MS * 16, n0 = tile.n * kTN;
    const int m_rows = min(MS * 16, a.M - m0), n_rows = min(kTN, a.N - n0);

    const int steps = a.K >> 7, NG = a.K / a.group, spg = a.group >> 7;
    const int s_begin = (wave * steps) / W, s_end = ((wave + 1) * steps) / W;
    const int n16 = (a.N + 15) >> 4;

    // ---- where the operands come from.  Rows and weight tiles past the end read the last one: what comes of them is
    // never stored.
    const int m16 = (a.M + 15) >> 4;
    const auto xres = buffer_of(a.xp, (size_t)m16 * steps * 2048);
    const auto wres = W8 ? xres : buffer_of(a.w, (size_t)n16 * steps * kPkBlockBytes);
    const auto sres = W8 ? buffer_of(a.scale, (size_t)a.N * NG * 4) : buffer_of(a.scale, (size_t)n16 * NG * 64);
    int x_off[MS], w_off[kNS], s_off[kNS];
#pragma unroll
    for (int i = 0; i < MS; ++i) x_off[i] = min((m0 >> 4) + i, m16 - 1) * steps * 2048 + lane * 16;
#pragma unroll
    for (int j = 0; j < kNS; ++j) {
        if constexpr (W8) {
            s_off[j] = min(n0 + 16 * j + li, a.N - 1) * NG * 4;
        } else {
            const int nt = min((n0 >> 4) + j, n16 - 1);
            w_off[j] = nt * steps * kPkBlockBytes + lane * 16;
            s_off[j] = nt * NG * 64 + li * 4;
        }
    }
    static_assert(!(W8 && WIDE), "int8 weights find wide scales themselves");
    v4i_t xa[MS][2], wr[kNS];
    int sc[kNS];
    auto load_x = [&](int i, int s) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            xa[i][h] = __builtin_amdgcn_raw_buffer_load_b128(xres, x_off[i] + h * 1024, s * 2048, 0);
    };
    auto load_w = [&](int s, int g) {
#pragma unroll
        for (int j = 0; j < kNS; ++j) {
            wr[j] = __builtin_amdgcn_raw_buffer_load_b128(wres, w_off[j], s * kPkBlockBytes, 0);
            sc[j] = __builtin_amdgcn_raw_buffer_load_b32(sres, s_off[j], g * 64, 0);
        }
    };
    // int8 weights are row-major: a load takes 8 whole 128-byte lines (one K step of 8 rows) straight to a stage of LDS that
    // belongs to the wave alone, and the operands are read from there (fetched to registers in 64-byte pieces every line
    // travelled twice: 300 x 4096 x 14336 131 us).  Two stages of 8 KB in the place of the wave's partial tile.  The 16-byte
    // chunks of a row are permuted by (row >> 1) & 7, so that the operand reads of 16 rows fall on different banks.
    const unsigned lds_stage = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem + wave * 2 * kStage8;
    v4i w8desc;
    int w8_off[8], w8_read[2];
    if constexpr (W8) {
        w8desc = make_desc(a.w, (size_t)a.N * a.K);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const int r = 8 * b + (lane >> 3);
            // (the load's own offset of 1024 (b & 3), which is meant for LDS, is taken off again here: where that is
            // negative, in a matrix of few short rows, the row is a repeated one, and reads as zero)
            w8_off[b] = min(n0 + r, a.N - 1) * a.K + (((lane & 7) ^ ((r >> 1) & 7)) << 4) - (b & 3) * 1024;
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) w8_read[h] = wave * 2 * kStage8 + li * 128 + (((4 * h + kb) ^ ((li >> 1) & 7)) << 4);
    }
    auto request_w8 = [&](int s) {
        const unsigned base = lds_stage + (s & 1) * kStage8;
        load_to_lds_rows_4x1k(w8desc, base, w8_off[0], w8_off[1], w8_off[2], w8_off[3], s * 128);
        load_to_lds_rows_4x1k(w8desc, base + 4096, w8_off[4], w8_off[5], w8_off[6], w8_off[7], s * 128);
    };
    // The scales of a weight row are contiguous along K: lane (li, kb) asks for that of K step s + kb, four steps at once.
    auto load_sc8 = [&](int s) {
        const int st = min(s + kb, steps - 1);
        const int g = spg == 1 ? st : st / spg;
#pragma unroll
        for (int j = 0; j < kNS; ++j) sc[j] = __builtin_amdgcn_raw_buffer_load_b32(sres, s_off[j] + g * 4, 0, 0);
    };

    using acc4 = typename std::conditional<INT_SCALE, v4i_t, v4f_t>::type;
    acc4 acc[MS][kNS];
    // (int8 weights: the largest and smallest integer scale met; the kernel layout of int4 weights says it in its header)
    int sc_max = 0, sc_min = 0;
    auto k_loop = [&](auto wide_c) {
        constexpr bool kWideNow = decltype(wide_c)::value;
#pragma unroll
        for (int i = 0; i < MS; ++i)
#pragma unroll
            for (int j = 0; j < kNS; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;
        if (s_begin >= s_end) return;  // (a K range of fewer steps than waves leaves some without any)
        auto correction = [&](int i) {
            v4i_t c = {0, 0, 0, 0};
            if constexpr (!W8) {
                constexpr int kM8 = (int)0xF8F8F8F8u;
                const v4i_t m8 = {kM8, kM8, kM8, kM8};
                c = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][0], m8, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][1], m8, c, 0, 0, 0);
            }
            return c;
        };
        auto scale_into = [&](acc4& dst, const v4i_t& part, int sc_i) {
            const float s_f = __int_as_float(sc_i);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if constexpr (!INT_SCALE) dst[r] = fmaf((float)part[r], s_f, dst[r]);  // C' += float(C_g) * s_g
                else if constexpr (kWideNow) {
                    int prod = part[r] * sc_i;
                    asm volatile("" : "+v"(prod));  // else a 64-bit multiply-add with register pairs
                    dst[r] += prod;
                } else dst[r] += __mul24(part[r], sc_i);  // C'' += C_g * s_g^INT
            }
        };
        int g = s_begin / spg, sub = s_begin - g * spg;
        int sc4[kNS];
        if constexpr (W8) {
            load_sc8(s_begin);
            request_w8(s_begin);
        } else {
            load_w(s_begin, g);
        }
#pragma unroll
        for (int i = 0; i < MS; ++i) load_x(i, s_begin);
        for (int s = s_begin; s < s_end; ++s) {
            const int next = min(s + 1, s_end - 1);  // (the last step asks for itself again: nobody uses it)
            if (s + 1 < s_end && ++sub == spg) {
                sub = 0;
                ++g;
            }
            v4i_t bu[kNS][2];
            int scl[kNS];
            if constexpr (W8) {
                const int t = (s - s_begin) & 3;
                if (t == 0) {
#pragma unroll
                    for (int j = 0; j < kNS; ++j) sc4[j] = sc[j];
                    load_sc8(s + 4);
                }
                // This step's lines are in LDS once at most the requests behind them are outstanding: the activations', and the
                // scales' just above.
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * MS) : "memory");
#pragma unroll
                for (int j = 0; j < kNS; ++j) {
                    scl[j] = __builtin_amdgcn_ds_bpermute((t * 16 + li) * 4, sc4[j]);
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        bu[j][h] = *reinterpret_cast<const v4i_t*>(smem + w8_read[h] + (s & 1) * kStage8 + j * 2048);
                }
            } else {
#pragma unroll
                for (int j = 0; j < kNS; ++j) {
                    scl[j] = sc[j];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const uint32_t pw = (uint32_t)wr[j][q];
                        bu[j][0][q] = (int)((pw ^ 0x08080808u) & 0x0F0F0F0Fu);         // k 0..63 of the step: low nibbles
                        bu[j][1][q] = (int)(((pw >> 4) ^ 0x08080808u) & 0x0F0F0F0Fu);  // k 64..127: high nibbles
                    }
                }
            }
            if constexpr (W8 && INT_SCALE && !kWideNow) {
                static_assert(kNS == 4, "two three-way maxima");
                sc_max = max(max(max(max(sc_max, scl[0]), scl[1]), scl[2]), scl[3]);
                sc_min = min(min(min(min(sc_min, scl[0]), scl[1]), scl[2]), scl[3]);
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (W8) request_w8(next);
            else load_w(next, g);
            __builtin_amdgcn_sched_barrier(0);
            v4i_t part[2][kNS];
            v4i_t ci = correction(0);
#pragma unroll
            for (int i = 0; i < MS; ++i) {
                const int cur = i & 1, prev = cur ^ 1;
#pragma unroll
                for (int j = 0; j < kNS; ++j)
                    part[cur][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][0], bu[j][0], ci, 0, 0, 0);
#pragma unroll
                for (int j = 0; j < kNS; ++j)
                    part[cur][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][1], bu[j][1], part[cur][j], 0, 0, 0);
                if (i + 1 < MS) ci = correction(i + 1);
                __builtin_amdgcn_sched_barrier(0);
                load_x(i, next);
                __builtin_amdgcn_sched_barrier(0);
                if (i > 0) {  // the scale step of the sub-tile before, under this one's MFMAs
#pragma unroll
                    for (int j = 0; j < kNS; ++j) scale_into(acc[i - 1][j], part[prev][j], scl[j]);
                }
            }
#pragma unroll
            for (int j = 0; j < kNS; ++j) scale_into(acc[MS - 1][j], part[(MS - 1) & 1][j], scl[j]);
        }
    };
    k_loop(std::integral_constant<bool, WIDE>{});
    if constexpr (W8 && INT_SCALE) {  // a scale of more than 24 signed bits was among them: once more, with full multiplies
        if (__any(sc_max >= (1 << 23) || sc_min < -(1 << 23))) k_loop(std::true_type{});
    }

    if constexpr (W8) {  // every wave is done with its stages, and nothing is on its way to them any more
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    }
    // ---- the waves' partial tiles meet in LDS: [wave][sub-tile i][j][lane][4 rows], 16 bytes a lane, no bank conflicts.
    // Units of one token sub-tile and two weight sub-tiles are dealt to the waves, which add them in wave order.
    v4i_t* parts = reinterpret_cast<v4i_t*>(smem);
    __half* otile = reinterpret_cast<__half*>(smem + sums_bytes(MS, W));
    constexpr int IC = rows_at_once(MS, W);
    const float inv_alpha = __int_as_float((127 - a.alpha_log2) << 23);
#pragma unroll
    for (int i0 = 0; i0 < MS; i0 += IC) {
        if (i0 > 0) __syncthreads();
#pragma unroll
        for (int ii = 0; ii < IC; ++ii)
#pragma unroll
            for (int j = 0; j < kNS; ++j) {
                if (i0 + ii >= MS) continue;
                v4i_t o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (INT_SCALE) o[r] = acc[(i0 + ii) % MS][j][r];
                    else o[r] = __float_as_int(acc[(i0 + ii) % MS][j][r]);
                }
                parts[((wave * IC + ii) * kNS + j) * kWave + lane] = o;
            }
        __syncthreads();
        constexpr int kUnits = IC * kNS / 2;
#pragma unroll
        for (int u0 = 0; u0 < kUnits; u0 += W) {
            const int u = u0 + wave;  // (uniform over the wave)
            if (u >= kUnits) break;
            const int ii = u / (kNS / 2), jp = u - ii * (kNS / 2), i = i0 + ii;
            if (i >= MS) break;
            acc4 v[2];
            float c[2], sa[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) sa[r] = a.a_scale[min(m0 + 16 * i + 4 * kb + r, a.M - 1)];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int nl = (2 * jp + j) * 16 + li;
                c[j] = 1.0f;
                if constexpr (INT_SCALE) {
                    if (a.chan_scale) c[j] = a.chan_scale[min(n0 + nl, a.N - 1)];
                    c[j] *= inv_alpha;
                }
                v4i_t got[W];
#pragma unroll
                for (int w = 0; w < W; ++w) got[w] = parts[((w * IC + ii) * kNS + 2 * jp + j) * kWave + lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (INT_SCALE) {
                        v[j][r] = got[0][r];
#pragma unroll
                        for (int w = 1; w < W; ++w) v[j][r] += got[w][r];
                    } else {
                        v[j][r] = __int_as_float(got[0][r]);
#pragma unroll
                        for (int w = 1; w < W; ++w) v[j][r] += __int_as_float(got[w][r]);
                    }
                }
                if constexpr (INT_SCALE) {
                    if (a.acc_out) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int ml = 16 * i + 4 * kb + r;
                            if (ml < m_rows && nl < n_rows) a.acc_out[(size_t)(m0 + ml) * a.N + n0 + nl] = v[j][r];
                        }
                    }
                }
            }
            // FLOAT(acc) * s_a[m] * c[n] / alpha (Eq. (2)), or facc * s_a[m] (Eq. (1))
            auto result = [&](int j, int r) {
                if constexpr (INT_SCALE) return __float2half_rn((float)v[j][r] * sa[r] * c[j]);
                else return __float2half_rn(v[j][r] * sa[r]);
            };
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                __half* row = otile + (16 * i + 4 * kb + r) * kPitch;
                if constexpr (SILU) {  // the two weight sub-tiles are the gate and up rows of the same 16 outputs
                    row[jp * 16 + li] = __float2half_rn(silu_mul(__half2float(result(0, r)), __half2float(result(1, r))));
                } else {
                    row[2 * jp * 16 + li] = result(0, r);
                    row[(2 * jp + 1) * 16 + li] = result(1, r);
                }
            }
        }
    }
    __syncthreads();
    const int out_n = SILU ? a.N >> 1 : a.N, out_n0 = SILU ? n0 >> 1 : n0, out_cols = SILU ? n_rows >> 1 : n_rows;
    constexpr int kCols = SILU ? kTN / 2 : kTN;
    __half* out = a.out + (size_t)m0 * out_n + out_n0;
    if ((out_n & 7) == 0) {  // 16 bytes a lane
        constexpr int kChunks = kCols / 8;
        for (int e = tid; e < MS * 16 * kChunks; e += W * kWave) {
            const int ml = e / kChunks, ch = e % kChunks;
            if (ml < m_rows && ch * 8 < out_cols)
                *reinterpret_cast<uint4*>(out + (size_t)ml * out_n + ch * 8) = *reinterpret_cast<const uint4*>(otile + ml * kPitch + ch * 8);
        }
    } else {
        for (int e = tid; e < MS * 16 * kCols; e += W * kWave) {
            const int ml = e / kCols, col = e % kCols;
            if (ml < m_rows && col < out_cols) out[(size_t)ml * out_n + col] = otile[ml * kPitch + col];
        }
    }
}

// (two waves per SIMD: 256 registers a wave, and MFMA results in ordinary registers, where the scale step reads them)
template <bool INT_SCALE, bool W8, int MS, int W, bool SILU>
__global__ __launch_bounds__(W* kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_wavek_kernel(WavekArgs a) {
    extern __shared__ __align__(16) unsigned char smem_wk[];
    if constexpr (INT_SCALE && !W8) {
        if (*reinterpret_cast<const int32_t*>(a.flags) & kPkFlagWide) {
            wavek_tile<true, true, false, MS, W, SILU>(a, smem_wk);
            return;
        }
    }
    wavek_tile<INT_SCALE, false, W8, MS, W, SILU>(a, smem_wk);
}

template <bool INT_SCALE, bool W8, int MS, int W, bool SILU>
hipError_t launch_instance(const WavekArgs& a, hipStream_t stream) {
    static LdsLimit limit;  // per instantiation
    auto kernel = gemm_wavek_kernel<INT_SCALE, W8, MS, W, SILU>;
    const hipError_t r = limit.raise(reinterpret_cast<const void*>(kernel), (int)lds_bytes(MS, W, W8));
    if (r != hipSuccess) return r;
    const long long tiles = (long long)((a.N + kTN - 1) / kTN) * ((a.M + MS * 16 - 1) / (MS * 16));
    hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(W * kWave), lds_bytes(MS, W, W8), stream, a);
    return hipGetLastError();
}

template <bool INT_SCALE, bool W8, bool SILU>
hipError_t launch_shape(const WavekArgs& a, const WavekPlan& p, hipStream_t stream) {
    if constexpr (!W8) {
        if (p.ms == 5 && p.waves == 8) return launch_instance<INT_SCALE, W8, 5, 8, SILU>(a, stream);
    }
    if (p.ms == 5) return launch_instance<INT_SCALE, W8, 5, 4, SILU>(a, stream);
    if (p.ms == 3) return p.waves == 8 ? launch_instance<INT_SCALE, W8, 3, 8, SILU>(a, stream) : launch_instance<INT_SCALE, W8, 3, 4, SILU>(a, stream);
    return p.waves == 8 ? launch_instance<INT_SCALE, W8, 4, 8, SILU>(a, stream) : launch_instance<INT_SCALE, W8, 4, 4, SILU>(a, stream);
}

}  // namespace

// A call's time with row tiles of 16 ms rows and workgroups of `waves`, in microseconds: launches, preparation and the like; per workgroup
// of a compute unit (four waves: two of them at a time) its start and end, and per K step of a wave a share by rows, with the SIMD to
// itself or shared; the weights' way from memory.  Fits of 96 calls with int4 and 60 with int8 weights, each with six plans (65 to 1000
// rows, 2048 to 28672 columns, K 4096 to 28672): 3 and 6 % off, and the best plan by them costs 0.4 and 0.5 % on average, 7 and 10 %
// at most.
static double wavek_us(int M, int N, int K, bool w8, int ms, int waves) {
    struct Fit {
        double call, end, end_rows, both, both_rows, alone, alone_rows, weights;
    };
    constexpr Fit kInt4{6.7, 0.88, 0.53, 0.23, 0.23, 0.27, 0.089, 0.0063}, kInt8{4.3, 0.65, 1.1, 0.93, 0.15, 0.77, 0.013, 0.13};
    const Fit& f = w8 ? kInt8 : kInt4;
    const long long tiles = (long long)((N + kTN - 1) / kTN) * ((M + ms * 16 - 1) / (ms * 16));
    const double per_cu = (double)((tiles + cu_count() - 1) / cu_count()), run = ((K >> 7) + waves - 1) / waves;
    const double ends = f.end + f.end_rows * ms, both = ends + run * (f.both + f.both_rows * ms), alone = ends + run * (f.alone + f.alone_rows * ms);
    const double pairs = floor(per_cu / 2);
    return f.call + (waves == 8 ? per_cu * both : pairs * both + (per_cu - 2 * pairs) * alone) + f.weights * 1e-6 * N * (double)K;
}

WavekPlan wavek_plan(int M, int N, int K, bool w8) {
    WavekPlan p;
    const auto tiles = [&](int ms) { return (long long)((N + kTN - 1) / kTN) * ((M + ms * 16 - 1) / (ms * 16)); };
    // row tiles of 48 or 64 rows, whichever pads less
    const int m16 = (M + 15) / 16;
    p.ms = (m16 + 2) / 3 * 3 < (m16 + 3) / 4 * 4 ? 3 : 4;
    p.tiles = tiles(p.ms);
    // Eight waves where workgroups of four would leave every compute unit with one wave per SIMD at most (65 x 4096 x 14336:
    // 22.1 against 24.0 us); two workgroups of four share a unit otherwise, one's start and end under the other's K loop.
    p.waves = p.tiles <= cu_count() ? 8 : 4;
    p.us = wavek_us(M, N, K, w8, p.ms, p.waves);
    // Long runs and more than a few tiles: by time, and tiles of 80 rows too.  What decides is how the tiles fill the units (300 x 4096: 320
    // tiles of 64 rows give a quarter of the 256 units two, 256 tiles of 80 rows give each one): W8A8 300 x 4096 x 14336 54.6 -> 42.4 us,
    // 400 rows 87 -> 58, 1024 rows 128 (tiled kernel) -> 108; int4 weights 300 x 4096 x 14336 41.9 -> 32.4, 200 rows 49.9 (tiled kernel) -> 27.8.
    if (K >= 2048 && p.tiles >= cu_count() / 8) {
        // The rule's tiles stay unless a twentieth is to be gained: near ties are decided by what the times leave out (173 x 15206 x 8064:
        // both 41.9 us by the times, 42.8 with 64 rows and 45.9 with 48).
        const double rule = p.us;
        for (int ms = 3; ms <= 5; ++ms)
            for (int waves = 4; waves <= (w8 && ms == 5 ? 4 : 8); waves += 4) {  // (80 rows of int8 weights: eight waves never ahead by these times)
                const double us = wavek_us(M, N, K, w8, ms, waves);
                if (us < p.us) {
                    p.us = us;
                    if (us < 0.95 * rule) {
                        p.ms = ms;
                        p.waves = waves;
                        p.by_padding = false;
                    }
                }
            }
        p.tiles = tiles(p.ms);
    }
    return p;
}

// This kernel's time against the tiled kernel's, in microseconds.  The tiled kernel with int4 weights: 20 us and 1.15 us per K step where a
// unit has one of its tiles at most (702 x 9559 x 2816 46 us, 1024 x 8192 x 8192 86, 512 x 16384 x 14336 144, 1024 x 8192 x 28672 286),
// 22 us and 1.62 us per step for two (762 x 12009 x 2048 50 us, 1000 x 12288 x 4096 72, 1000 x 10240 x 8192 124), and for few tiles, whose
// K range it cuts, 20 us to pass partial tiles through memory.  With one full round of the tiled kernel or more there are sixteen
// rounds of tiles here, and their starts and ends add up (540 x 53283 x 1536 97 us there, 108 us here; 4096 x 4608 x 2304 73 and 79 us; the
// best of such calls here is 3 % ahead).  4 % to spare with int4 weights: the long runs of large calls are slower than the fit says (1024 x 8192 x 28672
// 313 us here).  Where the two times are within 15 % and the tiles are those that pad least, a coarser time decides that counts rounds of
// 0.76 us per K step of a wave on every SIMD and was fitted to 1482 calls (wrong by 6 % at most near the line, the finer one by 8 %:
// 929 x 11092 x 2944 60.1 us here and 64.7 there, 946 x 11917 x 6784 108.3 and 113.9, 943 x 11445 x 4352 77.7 and 81.1).
static double tiled_us(long long tiles, int steps) {
    const int cus = cu_count();
    if (tiles > cus) return 22.0 + 1.62 * steps * (double)((tiles + 2 * cus - 1) / (2 * cus));
    const int parts = std::min(std::min(cus / (int)tiles, 8), std::max(steps / 8, 1));
    return 20.0 + (parts > 1 ? 1.56 * steps / parts : 1.15 * steps);
}

// With int8 weights the tiled kernel works on one tile per unit at a time, 1.03 us per K step, behind 9.5 us of launches and scale
// transposition; there the ends decide short K ranges, 2 us a round here and 10 us a tile there: 4096 x 4096 x 128 38 us here and 30 us there,
// 1109 x 719 x 384 11 and 20 us, 504 x 18148 x 1664 50 and 57 us; wide matrices are faster here than the fit says (104 x 24840 x 3712 46 and
// 54 us).
bool wavek_is_faster(int M, int N, int K, bool w8) {
    const int steps = K >> 7, cus = cu_count();
    const WavekPlan p = wavek_plan(M, N, K, w8);
    const long long tiles = (long long)((N + 255) / 256) * ((M + 127) / 128);
    double here = (w8 ? 0.95 : 1.04) * p.us;
    if (w8) {
        if (steps < 16) {  // (runs of a few steps a wave: by steps, not by the longest wave's)
            const double filled = std::max(1.0, 0.5 * ((double)((p.tiles + cus - 1) / cus) + (double)p.tiles / cus));
            here = 8.0 + filled * (2.0 + 0.72 * 0.25 * steps * (2 * p.ms + 8) / 12.0);
        }
        return here < 9.5 + (double)((tiles + cus - 1) / cus) * (10.0 + 1.03 * steps);
    }
    if (tiles >= 2 * cus) return false;
    double there = tiled_us(tiles, steps), tie = 0.15;
    if (steps < 16) {
        // Runs of a few steps a wave: rounds of tiles of which the last may be part filled, against starts that weigh more than steps (fits to
        // 1583 calls, 65 to 2100 rows, 256 to 40000 columns: 7 and 3 % off; with the coarser time for near ties the choice costs 0.1 % on
        // average and 11 % at most): 85 x 6496 x 256 8.4 us here and 15.7 there; 802 x 8064 x 512 24.3 and 20.7, 657 x 11968 x 512 27.7 and 24.5;
        // near ties: 300 x 27136 x 1664 38 and 41.
        const double rounds = std::max(1.0, 0.5 * ((double)((p.tiles + cus - 1) / cus) + (double)p.tiles / cus));
        here = 8.1 + rounds * (0.6 + 0.03 * p.ms + (steps + p.waves - 1) / p.waves * (0.155 + 0.106 * p.ms)) + 0.032e-6 * N * K;
        there = 12.95 + (tiles <= cus ? 0.77 + 1.1 * steps : 1.4 + 1.57 * steps);
        tie = 0.08;
    }
    if (!p.by_padding || here < (1.0 - tie) * there || here > (1.0 + tie) * there) return here < there;
    const double coarse = 10.0 + 0.76 * 0.25 * (double)((p.tiles + cus - 1) / cus) * steps * (2 * p.ms + 4) / 12.0;
    if (tiles > cus) return coarse < 6.0 + 2.3 * steps;
    const int parts = std::min(std::min(cus / (int)tiles, 8), std::max(steps / 8, 1));
    return coarse < 6.0 + (parts > 1 ? 1.56 * steps / parts + 14.0 : std::min(1.56 * steps, 25.0 + 1.31 * steps));
}

double prepared_gemm_us(int M, int N, int K) {
    const long long tiles = (long long)((N + 255) / 256) * ((M + 127) / 128);
    if (!wavek_is_faster(M, N, K, false)) return tiled_us(tiles, K >> 7);
    return wavek_plan(M, N, K, false).us;
}

void wavek_kernel_name(const WavekPlan& p, bool int_scale, bool w8, bool silu, char* buf, size_t len) {
    snprintf(buf, len, "gemm_wavek_kernel<%s, %s, %d, %d, %s>", int_scale ? "true" : "false", w8 ? "true" : "false", p.ms, p.waves,
             silu ? "true" : "false");
}

hipError_t launch_gemm_wavek(const WavekArgs& a, const WavekPlan& p, bool int_scale, bool w8, bool silu, hipStream_t stream) {
    if (w8) return int_scale ? launch_shape<true, true, false>(a, p, stream) : launch_shape<false, true, false>(a, p, stream);
    if (silu) return int_scale ? launch_shape<true, false, true>(a, p, stream) : launch_shape<false, false, true>(a, p, stream);
    return int_scale ? launch_shape<true, false, false>(a, p, stream) : launch_shape<false, false, false>(a, p, stream);
}

}  // namespace intscale
