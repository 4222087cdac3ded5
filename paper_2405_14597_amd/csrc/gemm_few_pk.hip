// Fine-grained W4A8 GEMM on prepacked weights, 1 to 64 token rows (and, in row tiles, calls of up to 512; and experts of few rows): the
// waves of a workgroup split K.
// Integer-scale form: Eq. (2) / Table 2 "Ours" of the Integer Scale paper; float-scale form: Eq. (1) / Table 2 "Atom".
// (An fp16 row, a float-scale row, a quantised row with a long K, and narrow matrices with a long K have a kernel of their own,
// gemm_decode_pk.hip.)
//
// What bounds this regime: the weight stream from memory where the matrix is large and the rows are few, the kernel's start and end
// where it is small.  With 64 rows a compute unit mostly has one workgroup of four waves, one a SIMD, which issues 46 % of its time,
// waits for loads 31 % and for an issue slot 23 %; the matrix pipe is busy a fifth of the time and the L2 delivers 19 bytes a
// cycle and unit where it can 45 to 55 (64 x 12288 x 4096, 11.2 us; 9.4 without the loads of the activations, 8 KB a K step next to 1 KB
// per weight tile).  So a workgroup takes a few 16-row weight tiles and all of K,
// each of its 4 or 8 waves multiplies all of them over its own run of K steps, and the partial sums meet once, in LDS: no barrier in
// the loop, no partial tile leaves the compute unit, nothing waits for the activations of a whole slab (a kernel that keeps
// them in LDS for all its waves cuts K over workgroups where they do not fit, and the partial tiles then travel through memory).
//
// Operands.  Weights go from the kernel layout straight to registers, a contiguous kilobyte a load, D K steps ahead.  Activations
// are read in their canonical row-major layout (no preparation kernel): a load takes 8 whole 128-byte lines straight to a stage of LDS
// that belongs to the wave alone, two steps ahead, with the 16-byte chunks of a row permuted by (row >> 1) & 7 so that the operand
// reads of 16 rows fall on different banks.  A wave's loads return in order, so the waits count requests.
//
// int4 -> int8 with a zero point: (word ^ 0x08..) & 0x0F.. is q + 8, and every MFMA chain starts from -8 sum_k x[m,k], which the matrix
// pipe gives itself (a multiplication by a constant operand of -8s, once per step for all weight tiles).
//
// Measured (GEMM on int8 codes, graph replay, cold weights, N x K; the kernel with the activations in LDS and K cut over
// workgroups first): 16 rows: 4096 x 4096 6.5 -> 5.0 us, 12288 x 4096 8.2 -> 7.3, 4096 x 11008 10.1 -> 7.5, 57344 x 8192 49.5 -> 45.6;
// 32 rows: 4096 x 4096 9.0 -> 5.7, 22016 x 4096 14.9 -> 13.0, 57344 x 8192 63 -> 51, 8192 x 28672 32.8 -> 33.5; 64 rows: 4096 x 4096
// 11.1 -> 7.3, 12288 x 4096 15.9 -> 10.3, 22016 x 4096 24.3 -> 18.7, 10240 x 8192 22.8 -> 17.2; on 359 calls 0.77 of its time.
#include <math.h>
#include <stdio.h>

#include <algorithm>

#include "act_common.h"
#include "few_common.h"
#include "pk_common.h"
#include "tile_common.h"

namespace intscale {
namespace {

typedef int v4i_t __attribute__((ext_vector_type(4)));
typedef float v4f_t __attribute__((ext_vector_type(4)));

constexpr int kOutOfRange = (int)0x80000000u;  // a buffer offset past every descriptor here

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}

// Sub-tiles of token rows whose partial sums pass through LDS at a time
constexpr int rows_at_once(int MS, int NS, int W) {
    int c = MS;
    while ((size_t)W * c * NS * 1024 > 112 * 1024) c = (c + 1) / 2;
    return c;
}
constexpr size_t stage_area(int MS, int NS, int W) {
    const size_t stages = (size_t)W * 2 * MS * 2048, sums = (size_t)W * rows_at_once(MS, NS, W) * NS * 1024;
    return stages > sums ? stages : sums;
}
constexpr int out_pitch(int NS) { return NS * 16 + 8; }
constexpr size_t few_lds_bytes(int MS, int NS, int W) {
    return stage_area(MS, NS, W) + (size_t)MS * 16 * out_pitch(NS) * 2 + 256 + 512;
}

// What a workgroup works on: `m_rows` (at most 16 MS) token rows and NS 16-row weight tiles from `t0` on, over all of K.
struct FewTile {
    const int8_t* x;          // its first token row
    const float* a_scale;
    const uint8_t* wpack;
    const uint8_t* spack;
    const float* chan_scale;
    __half* out;              // its first token row's outputs
    int32_t* acc_out;
    int m_rows, t0;
    int phase;                // differs between the workgroups of an XCD
};

template <bool INT_SCALE, int MS, int NS, int W, int D, bool SILU>
__device__ __forceinline__ void few_tile(const FewArgs& a, const FewTile& t, unsigned char* smem) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int li = lane & 15, kb = lane >> 4;
    // ("some integer scale needs more than 24 signed bits": asked for here, needed behind the first requests)
    const int flags = *reinterpret_cast<const int32_t*>(t.spack);
    const int steps = a.K >> 7, NG = a.num_groups, spg = a.group >> 7;
    const int s_begin = (wave * steps) / W, s_end = ((wave + 1) * steps) / W;
    // Where the wave starts in its run of K steps differs from workgroup to workgroup (it goes round): rows a power of two apart
    // lie on one channel of the L2, and in step all workgroups would read the same few of them.
    const int s_first = s_begin + (t.phase & a.phase_mask);
    const int n16 = (a.N + 15) >> 4, n0 = t.t0 * 16;

    // ---- token scales and channel scales to LDS, in front of everything else
    constexpr size_t kOtile = stage_area(MS, NS, W), kAux = kOtile + (size_t)MS * 16 * out_pitch(NS) * 2;
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    auto load_words = [&](const void* base, unsigned words, unsigned at) {  // 64 words, zeros past the end
        const v4i d = make_desc(base, (size_t)words * 4);
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds0 + at), "v"(lane * 4), "s"(d) : "memory");
    };
    if (wave == 0) {
        load_words(t.a_scale, t.m_rows, kAux);
        if constexpr (INT_SCALE) {
            if (t.chan_scale) {
                load_words(t.chan_scale + n0, a.N - n0, kAux + 256);
                if constexpr (NS > 4) load_words(t.chan_scale + min(n0 + 64, a.N), max(a.N - n0 - 64, 0), kAux + 512);
            }
        }
    }

    // ---- where the operands come from
    const unsigned wbytes = (unsigned)(n16 - t.t0) * (unsigned)steps * kPkBlockBytes, sbytes = (unsigned)(n16 - t.t0) * (unsigned)NG * 64;
    const uint8_t* wbase = t.wpack + (size_t)t.t0 * steps * kPkBlockBytes;
    const uint8_t* sbase = t.spack + kPkHeaderBytes + (size_t)t.t0 * NG * 64;
    int w_off[NS], s_off[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
        w_off[j] = j * steps * kPkBlockBytes + lane * 16;
        s_off[j] = j * NG * 64 + li * 4;
    }
    const unsigned xbytes = (unsigned)t.m_rows * (unsigned)a.K;
    v4i xdesc = make_desc(t.x, xbytes);
    int x_off[2 * MS];
#pragma unroll
    for (int b = 0; b < 2 * MS; ++b) {
        const int r = 8 * b + (lane >> 3);
        x_off[b] = r < t.m_rows ? r * a.K + (((lane & 7) ^ ((r >> 1) & 7)) << 4) - (b & 3) * 1024 : kOutOfRange;
    }
    const unsigned lds_stage = lds0 + wave * 2 * MS * 2048;
    int x_read[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) x_read[h] = wave * 2 * MS * 2048 + li * 128 + (((4 * h + kb) ^ ((li >> 1) & 7)) << 4);

    const int count = s_end - s_begin;  // the wave's K steps
    int x_at;                           // the one whose activations are asked for next
    auto request_x = [&](int slot, int i) {
        v4i d = xdesc;
        d[2] = i < count ? (int)xbytes : 0;  // (past the wave's last step: nothing is fetched, zeros are written)
        const int s = x_at;
        x_at = s + 1 == s_end ? s_begin : s + 1;
        const unsigned base = lds_stage + slot * MS * 2048;
        if constexpr (MS == 1) {
            load_to_lds_rows_2x1k(d, base, x_off[0], x_off[1], s * 128);
        } else {
            load_to_lds_rows_4x1k(d, base, x_off[0], x_off[1], x_off[2], x_off[3], s * 128);
            if constexpr (MS == 3) load_to_lds_rows_2x1k(d, base + 4096, x_off[4], x_off[5], s * 128);
            if constexpr (MS == 4) load_to_lds_rows_4x1k(d, base + 4096, x_off[4], x_off[5], x_off[6], x_off[7], s * 128);
        }
    };
    v4i_t wr[D][NS];
    int sc[D][NS];
    int w_at;  // the step whose weights are asked for next, and its group
    auto group_of = [&](int s) { return spg == 1 ? s : __builtin_amdgcn_readfirstlane(s / spg); };
    const int g_begin = group_of(s_begin), sub_begin = s_begin - g_begin * spg;
    int g_at, sub_at;
    auto request_w = [&](int slot, int j, int i) {
        const bool ok = i < count;
        const int s = w_at, g = g_at;
        wr[slot][j] = __builtin_amdgcn_raw_buffer_load_b128(buffer_of(wbase, ok ? wbytes : 0), w_off[j], s * kPkBlockBytes, 0);
        sc[slot][j] = __builtin_amdgcn_raw_buffer_load_b32(buffer_of(sbase, ok ? sbytes : 0), s_off[j], __builtin_amdgcn_readfirstlane(g * 64), 0);
    };

    using acc4 = typename std::conditional<INT_SCALE, v4i_t, v4f_t>::type;
    acc4 acc[MS][NS];
#pragma unroll
    for (int i = 0; i < MS; ++i)
#pragma unroll
        for (int j = 0; j < NS; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0;
    auto scale_into = [&](auto wide_c, acc4& dst, const v4i_t& part, int sc_i) {
        constexpr bool WIDE = decltype(wide_c)::value;
        const float s_f = __int_as_float(sc_i);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (!INT_SCALE) dst[r] = fmaf((float)part[r], s_f, dst[r]);  // C' += float(C_g) * s_g
            else if constexpr (WIDE) {
                int prod = part[r] * sc_i;
                asm volatile("" : "+v"(prod));  // else a 64-bit multiply-add with register pairs
                dst[r] += prod;
            } else dst[r] += __mul24(part[r], sc_i);  // C'' += C_g * s_g^INT
        }
        // (else the products of two steps meet in one three-way addition, and the first one's wait for it in registers)
        asm("" : "+v"(dst));
    };

    auto next_w = [&]() {
        const bool wrap = w_at + 1 == s_end, group_done = sub_at + 1 == spg;
        g_at = wrap ? g_begin : g_at + (group_done ? 1 : 0);
        sub_at = wrap ? sub_begin : group_done ? 0 : sub_at + 1;
        w_at = wrap ? s_begin : w_at + 1;
    };
    // One K step, in ring slot SLOT
    auto step = [&](auto wide_c, auto slot_c, int i_step) {
        constexpr int slot = decltype(slot_c)::value, xslot = slot & 1;
        constexpr bool kWide = decltype(wide_c)::value;
        __builtin_amdgcn_sched_barrier(0);  // (nothing of this step under the one before: it would not fit the registers)
#pragma unroll
        for (int j = 0; j < NS; ++j) asm volatile("" ::"v"(wr[slot][j]), "v"(sc[slot][j]));  // its weights have come
        // its activations as well: asked for two steps ago, younger are the next step's and the weights of the two steps behind each
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * NS + 2 * MS) : "memory");
        v4i_t xa[MS][2];
#pragma unroll
        for (int i = 0; i < MS; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) xa[i][h] = *reinterpret_cast<const v4i_t*>(smem + x_read[h] + xslot * MS * 2048 + i * 2048);
        v4i_t bu[2];
        auto unpack = [&](int j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t pw = (uint32_t)wr[slot][j][q];
                bu[0][q] = (int)((pw ^ 0x08080808u) & 0x0F0F0F0Fu);         // k 0..63 of the step: low nibbles
                bu[1][q] = (int)(((pw >> 4) ^ 0x08080808u) & 0x0F0F0F0Fu);  // k 64..127: high nibbles
            }
        };
        unpack(0);
        // (the operands are in registers: their place in LDS may be written again)
#pragma unroll
        for (int i = 0; i < MS; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(xa[i][0]), "+v"(xa[i][1])::"memory");
        request_x(xslot, i_step + 2);
        __builtin_amdgcn_sched_barrier(0);
        v4i_t ci[MS];
        constexpr int kM8 = (int)0xF8F8F8F8u;
        const v4i_t m8 = {kM8, kM8, kM8, kM8};
#pragma unroll
        for (int i = 0; i < MS; ++i) ci[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][0], m8, v4i_t{0, 0, 0, 0}, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < MS; ++i) ci[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][1], m8, ci[i], 0, 0, 0);
        v4i_t part[2][MS];
        int scl[2];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int cur = j & 1, prev = cur ^ 1;
            if (j > 0) unpack(j);
            // (a copy the compiler cannot look through: with the old scale still in use, the new one would be loaded elsewhere
            // and moved back at the end of the loop, behind a wait for the whole ring)
            asm volatile("v_mov_b32 %0, %1" : "=v"(scl[cur]) : "v"(sc[slot][j]));
            __builtin_amdgcn_sched_barrier(0);
            request_w(slot, j, i_step + D);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < MS; ++i) part[cur][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][0], bu[0], ci[i], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < MS; ++i) part[cur][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa[i][1], bu[1], part[cur][i], 0, 0, 0);
            if constexpr (kWide) {  // (at once: the full multiplies leave no registers for a second set of results)
#pragma unroll
                for (int i = 0; i < MS; ++i) scale_into(wide_c, acc[i][j], part[cur][i], scl[cur]);
                __builtin_amdgcn_sched_barrier(0);
            } else if (j > 0) {  // the scale step of the sub-tile before, under this one's MFMAs
#pragma unroll
                for (int i = 0; i < MS; ++i) scale_into(wide_c, acc[i][j - 1], part[prev][i], scl[prev]);
            }
        }
        next_w();
        if constexpr (!kWide) {
#pragma unroll
            for (int i = 0; i < MS; ++i) scale_into(wide_c, acc[i][NS - 1], part[(NS - 1) & 1][i], scl[(NS - 1) & 1]);
        }
    };
    auto first_requests = [&]() {
        x_at = w_at = s_first;
        g_at = group_of(s_first);
        sub_at = s_first - g_at * spg;
#pragma unroll
        for (int u = 0; u < D; ++u) {
            if (u < 2) request_x(u, u);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < NS; ++j) request_w(u, j, u);
            __builtin_amdgcn_sched_barrier(0);
            next_w();
        }
    };
    if (count > 0) {
        first_requests();
        // D steps a turn without a way out between them: behind one the compiler would wait for the ring's youngest loads.  (Steps
        // past the wave's last multiply zeros.)
        auto k_loop = [&](auto wide_c) {
            for (int i = 0; i < count; i += D) {
                step(wide_c, std::integral_constant<int, 0>{}, i);
                step(wide_c, std::integral_constant<int, 1>{}, i + 1);
                if constexpr (D == 4) {
                    step(wide_c, std::integral_constant<int, 2>{}, i + 2);
                    step(wide_c, std::integral_constant<int, 3>{}, i + 3);
                }
            }
        };
        if (INT_SCALE && (flags & kPkFlagWide) != 0) {
            // (asked for once more: one ring that both loops could begin with does not fit the registers.  The waits are the
            // compiler's own, so that it does not carry what is outstanding here into the other loop.)
            __builtin_amdgcn_s_waitcnt(0);
            first_requests();
            k_loop(std::true_type{});
            __builtin_amdgcn_s_waitcnt(0);
        } else {
            k_loop(std::false_type{});
        }
    }

    // ---- the waves' partial tiles meet in LDS (nothing is on its way to the stages any more)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    constexpr int IC = rows_at_once(MS, NS, W), kPitch = out_pitch(NS), JP = NS % 2 == 0 ? 2 : 1;
    static_assert(!SILU || JP == 2, "gate and up sub-tiles come in pairs");
    v4i_t* parts = reinterpret_cast<v4i_t*>(smem);
    __half* otile = reinterpret_cast<__half*>(smem + kOtile);
    const float* aux = reinterpret_cast<const float*>(smem + kAux);
    const float inv_alpha = __int_as_float((127 - a.alpha_log2) << 23);
    const int n_rows = min(NS * 16, a.N - n0);
#pragma unroll
    for (int i0 = 0; i0 < MS; i0 += IC) {
        if (i0 > 0) __syncthreads();
#pragma unroll
        for (int ii = 0; ii < IC; ++ii)
#pragma unroll
            for (int j = 0; j < NS; ++j) {
                if (i0 + ii >= MS) continue;
                v4i_t o;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if constexpr (INT_SCALE) o[r] = acc[(i0 + ii) % MS][j][r];
                    else o[r] = __float_as_int(acc[(i0 + ii) % MS][j][r]);
                }
                parts[((wave * IC + ii) * NS + j) * kWave + lane] = o;
            }
        __syncthreads();
        constexpr int kUnits = IC * NS / JP;
#pragma unroll
        for (int u0 = 0; u0 < kUnits; u0 += W) {
            const int u = u0 + wave;  // (uniform over the wave)
            if (u >= kUnits) break;
            const int ii = u / (NS / JP), jp = u - ii * (NS / JP), i = i0 + ii;
            if (i >= MS) break;
            acc4 v[JP];
            float c[JP];
            const v4f_t sa = *reinterpret_cast<const v4f_t*>(aux + 16 * i + 4 * kb);
#pragma unroll
            for (int j = 0; j < JP; ++j) {
                const int nl = (JP * jp + j) * 16 + li;
                c[j] = 1.0f;
                if constexpr (INT_SCALE) {
                    if (t.chan_scale) c[j] = aux[64 + nl];
                    c[j] *= inv_alpha;
                }
                v4i_t got[W];
#pragma unroll
                for (int w = 0; w < W; ++w) got[w] = parts[((w * IC + ii) * NS + JP * jp + j) * kWave + lane];
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
                    if (t.acc_out) {
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int ml = 16 * i + 4 * kb + r;
                            if (ml < t.m_rows && nl < n_rows) t.acc_out[(size_t)ml * a.N + n0 + nl] = v[j][r];
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
#pragma unroll
                    for (int j = 0; j < JP; ++j) row[(JP * jp + j) * 16 + li] = result(j, r);
                }
            }
        }
    }
    __syncthreads();
    const int out_n = SILU ? a.N >> 1 : a.N, out_n0 = SILU ? n0 >> 1 : n0, out_cols = SILU ? n_rows >> 1 : n_rows;
    constexpr int kCols = SILU ? NS * 8 : NS * 16;
    __half* out = t.out + out_n0;
    if ((out_n & 7) == 0) {  // 16 bytes a lane
        constexpr int kChunks = kCols / 8;
        for (int e = tid; e < t.m_rows * kChunks; e += W * kWave) {
            const int ml = e / kChunks, ch = e % kChunks;
            if (ch * 8 < out_cols)
                *reinterpret_cast<uint4*>(out + (size_t)ml * out_n + ch * 8) = *reinterpret_cast<const uint4*>(otile + ml * kPitch + ch * 8);
        }
    } else {
        for (int e = tid; e < t.m_rows * kCols; e += W * kWave) {
            const int ml = e / kCols, col = e % kCols;
            if (col < out_cols) out[(size_t)ml * out_n + col] = otile[ml * kPitch + col];
        }
    }
}

// (two waves per SIMD: 256 registers a wave, and MFMA results in ordinary registers, where the scale step reads them)
template <int MS, int NS, int W, int D, bool INT_SCALE, bool SILU>
__global__ __launch_bounds__(W* kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_few_pk_kernel(FewArgs a) {
    extern __shared__ __align__(16) unsigned char smem_few[];
    FewTile t;
    t.x = a.xq;
    t.a_scale = a.a_scale;
    t.wpack = a.wpack;
    t.spack = a.spack;
    t.chan_scale = a.chan_scale;
    t.out = a.out;
    t.acc_out = a.acc_out;
    t.m_rows = a.M;
    t.t0 = blockIdx.x * NS;
    t.phase = blockIdx.x / 16;
    few_tile<INT_SCALE, MS, NS, W, D, SILU>(a, t, smem_few);
}

// The launch's own arguments: groups along K, and the largest 2^n - 1 below the shortest wave's number of steps
FewArgs with_launch_arguments(const FewArgs& a, int waves) {
    FewArgs b = a;
    b.num_groups = a.K / a.group;
    b.phase_mask = 0;
    while (2 * b.phase_mask + 2 <= (a.K >> 7) / waves) b.phase_mask = 2 * b.phase_mask + 1;
    return b;
}

template <bool INT_SCALE, int MS, int NS, int W, int D, bool SILU>
hipError_t launch_instance(const FewArgs& a, hipStream_t stream) {
    static LdsLimit limit;  // per instantiation
    auto kernel = gemm_few_pk_kernel<MS, NS, W, D, INT_SCALE, SILU>;
    constexpr size_t lds = few_lds_bytes(MS, NS, W);
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    const hipError_t r = limit.raise(reinterpret_cast<const void*>(kernel), (int)lds);
    if (r != hipSuccess) return r;
    const int n16 = (a.N + 15) / 16;
    hipLaunchKernelGGL(kernel, dim3((n16 + NS - 1) / NS), dim3(W * kWave), lds, stream, with_launch_arguments(a, W));
    return hipGetLastError();
}

// Moderate numbers of rows, integer scales (exact in any order; float sums have to be those of the calls on prepared activations, bit for
// bit): the workgroups of several row tiles.
template <int MS, int NS, int W, int D, bool SILU>
__global__ __launch_bounds__(W* kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_rows_pk_kernel(FewArgs a) {
    extern __shared__ __align__(16) unsigned char smem_few[];
    const int tiles_n = (a.N + NS * 16 - 1) / (NS * 16), tiles_m = (a.M + MS * 16 - 1) / (MS * 16);
    const TileAt tile = tile_of_block(blockIdx.x, tiles_m, tiles_n);
    const int m0 = tile.m * MS * 16;
    FewTile t;
    t.x = a.xq + (size_t)m0 * a.K;
    t.a_scale = a.a_scale + m0;
    t.wpack = a.wpack;
    t.spack = a.spack;
    t.chan_scale = a.chan_scale;
    t.out = a.out + (size_t)m0 * (SILU ? a.N >> 1 : a.N);
    t.acc_out = a.acc_out ? a.acc_out + (size_t)m0 * a.N : nullptr;
    t.m_rows = min(a.M - m0, MS * 16);
    t.t0 = tile.n * NS;
    t.phase = tile.n / 2;
    few_tile<true, MS, NS, W, D, SILU>(a, t, smem_few);
}

// The nth of the row tiles (`rows_a_tile` rows) that experts have beside their first, by expert; false past the last one.  Uniform over
// the wave, 64 experts at a time, a lane each.
__device__ __forceinline__ bool further_tile(const FewGroups& g, int M, int rows_a_tile, int nth, int& expert, int& tile) {
    const int lane = threadIdx.x & (kWave - 1);
    for (int e0 = 0, base = 0; e0 < g.num_experts; e0 += kWave) {
        const int e = e0 + lane;
        const int rows = e < g.num_experts ? min(g.row_offsets[e + 1], M) - max(g.row_offsets[e], 0) : 0;
        const int further = rows > 0 ? (rows - 1) / rows_a_tile : 0;
        if (__ballot(further > 0) == 0) continue;
        const int upto = base + lanes_up_to(further, lane);
        const unsigned long long past = __ballot(nth < upto);
        if (past != 0) {
            const int who = __builtin_ctzll(past);
            expert = __builtin_amdgcn_readfirstlane(e0 + who);
            tile = __builtin_amdgcn_readfirstlane(nth - __shfl(upto - further, who, kWave) + 1);
            return true;
        }
        base = __builtin_amdgcn_readfirstlane(__shfl(upto, kWave - 1, kWave));
    }
    return false;
}

// Mixture-of-experts form: workgroup (x, y) takes NS weight tiles of an expert and 16 MT of its rows at a time: the first E along y the
// first rows of expert y (an expert without rows costs a workgroup's start), the others share what rows there are beyond them, so that an
// expert that many rows come to has many workgroups at work (in turns of one workgroup, 64 experts of 2816 x 2048 and all 1536 rows at
// one: #O us, #N this way; the tiled kernel 37).
struct FewGroupedArgs {
    FewArgs a;
    FewGroups g;
};

template <class T>
__device__ __forceinline__ T* in_global(T* p) { return (T*)(__attribute__((address_space(1))) T*)p; }

// The kernel's only argument read once more, in a way that the compiler cannot see through: a loop that reads it so each time keeps nothing
// of it alive.  (What it kept otherwise took 70 to 100 scalar registers more than there are, and scratch memory in two instances.)
__device__ __forceinline__ FewGroupedArgs arguments_again() {
    typedef __attribute__((address_space(4))) const FewGroupedArgs* args_t;
    args_t p = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    FewGroupedArgs r;
    r.a.xq = in_global(p->a.xq);
    r.a.a_scale = in_global(p->a.a_scale);
    r.a.wpack = in_global(p->a.wpack);
    r.a.spack = in_global(p->a.spack);
    r.a.chan_scale = in_global(p->a.chan_scale);
    r.a.out = in_global(p->a.out);
    r.a.acc_out = in_global(p->a.acc_out);
    r.a.M = p->a.M;
    r.a.N = p->a.N;
    r.a.K = p->a.K;
    r.a.group = p->a.group;
    r.a.alpha_log2 = p->a.alpha_log2;
    r.a.num_groups = p->a.num_groups;
    r.a.phase_mask = p->a.phase_mask;
    r.g.row_offsets = in_global(p->g.row_offsets);
    r.g.num_experts = p->g.num_experts;
    r.g.wstride = p->g.wstride;
    r.g.sstride = p->g.sstride;
    return r;
}

// Rows m to hi of expert e, 16 MT of them at most
template <int MT, int NS, int W, int D, bool INT_SCALE>
__device__ __forceinline__ void few_rows_of_expert(const FewGroupedArgs& p, int e, int m, int hi, unsigned char* smem) {
    const FewArgs& a = p.a;
    FewTile t;
    t.wpack = a.wpack + e * p.g.wstride;
    t.spack = a.spack + e * p.g.sstride;
    t.chan_scale = a.chan_scale ? a.chan_scale + (size_t)e * a.N : nullptr;
    t.t0 = blockIdx.x * NS;
    t.phase = blockIdx.x / 16;
    t.x = a.xq + (size_t)m * a.K;
    t.a_scale = a.a_scale + m;
    t.out = a.out + (size_t)m * a.N;
    t.acc_out = a.acc_out ? a.acc_out + (size_t)m * a.N : nullptr;
    t.m_rows = min(hi - m, 16 * MT);
    if constexpr (MT >= 4) {
        if (t.m_rows > 32) return few_tile<INT_SCALE, 4, NS, W, D, false>(a, t, smem);
    }
    if constexpr (MT >= 2) {
        if (t.m_rows > 16) return few_tile<INT_SCALE, 2, NS, W, D, false>(a, t, smem);
    }
    few_tile<INT_SCALE, 1, NS, W, D, false>(a, t, smem);
}

template <int MT, int NS, int W, int D, bool INT_SCALE>
__global__ __launch_bounds__(W* kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void gemm_few_grouped_pk_kernel(FewGroupedArgs args) {
    extern __shared__ __align__(16) unsigned char smem_few[];
    const int E = args.g.num_experts;
    if ((int)blockIdx.y < E) {  // (apart from the loop below, whose live values cost these 4 % of 8 x 28672 x 4096)
        const int m = max(args.g.row_offsets[blockIdx.y], 0), hi = min(args.g.row_offsets[blockIdx.y + 1], args.a.M);
        if (m < hi) few_rows_of_expert<MT, NS, W, D, INT_SCALE>(args, blockIdx.y, m, hi, smem_few);
        return;
    }
    int e = 0, tile = 0;
    for (int nth = blockIdx.y - E;;) {
        const FewGroupedArgs p = arguments_again();
        if (!further_tile(p.g, p.a.M, 16 * MT, nth, e, tile)) return;
        const int m = __builtin_amdgcn_readfirstlane(max(p.g.row_offsets[e], 0) + tile * 16 * MT);
        few_rows_of_expert<MT, NS, W, D, INT_SCALE>(p, e, m, __builtin_amdgcn_readfirstlane(min(p.g.row_offsets[e + 1], p.a.M)), smem_few);
        __syncthreads();  // the output tile has been read
        nth += gridDim.y - p.g.num_experts;
    }
}

template <int MS, int NS, bool SILU>
hipError_t launch_rows_instance(const FewArgs& a, hipStream_t stream) {
    static LdsLimit limit;  // per instantiation
    constexpr int W = 4;
    auto kernel = gemm_rows_pk_kernel<MS, NS, W, 2, SILU>;
    constexpr size_t lds = few_lds_bytes(MS, NS, W);
    const hipError_t r = limit.raise(reinterpret_cast<const void*>(kernel), (int)lds);
    if (r != hipSuccess) return r;
    const int tiles_n = (a.N + NS * 16 - 1) / (NS * 16), tiles_m = (a.M + MS * 16 - 1) / (MS * 16);
    hipLaunchKernelGGL(kernel, dim3(tiles_n * tiles_m), dim3(W * kWave), lds, stream, with_launch_arguments(a, W));
    return hipGetLastError();
}

template <int MT, int NS, int W, int D, bool INT_SCALE>
hipError_t launch_grouped_instance(const FewArgs& a, const FewGroups& g, hipStream_t stream) {
    static LdsLimit limit;  // per instantiation
    auto kernel = gemm_few_grouped_pk_kernel<MT, NS, W, D, INT_SCALE>;
    constexpr size_t lds = few_lds_bytes(MT, NS, W);
    const hipError_t r = limit.raise(reinterpret_cast<const void*>(kernel), (int)lds);
    if (r != hipSuccess) return r;
    // beside the experts' first tiles: as many workgroups as the chip holds at a time, or as there can be further tiles
    const int wgs = ((a.N + 15) / 16 + NS - 1) / NS, further = std::min((a.M - 1) / (16 * MT), (2 * cu_count() + wgs - 1) / wgs);
    hipLaunchKernelGGL(kernel, dim3(wgs, g.num_experts + further), dim3(W * kWave), lds, stream, FewGroupedArgs{with_launch_arguments(a, W), g});
    return hipGetLastError();
}

// The instances there are (few_plan chooses among them).  Four waves: up to as many weight tiles as the registers hold.  Eight: up
// to three (each compute unit then has one workgroup, and more tiles mean fewer of them).  Rings of four for long runs only.
constexpr bool has_instance(int ms, int ns, int waves, int depth, bool silu) {
    if (silu && ns % 2 != 0) return false;
    if (depth == 4) return ms <= 2 && (ns == 2 || (ns == 1 && waves == 8));
    if (waves == 8) return ns <= 3;
    return ns <= (ms == 1 ? 7 : ms == 2 ? 6 : ms == 3 ? 5 : 4);
}

template <bool INT_SCALE, bool SILU, int MS, int NS>
hipError_t launch_waves(const FewArgs& a, const FewPlan& p, hipStream_t stream) {
    if (p.waves == 4 && p.depth == 2) {
        if constexpr (has_instance(MS, NS, 4, 2, SILU)) return launch_instance<INT_SCALE, MS, NS, 4, 2, SILU>(a, stream);
    } else if (p.waves == 8 && p.depth == 2) {
        if constexpr (has_instance(MS, NS, 8, 2, SILU)) return launch_instance<INT_SCALE, MS, NS, 8, 2, SILU>(a, stream);
    } else if (p.waves == 4 && p.depth == 4) {
        if constexpr (has_instance(MS, NS, 4, 4, SILU)) return launch_instance<INT_SCALE, MS, NS, 4, 4, SILU>(a, stream);
    } else if (p.waves == 8 && p.depth == 4) {
        if constexpr (has_instance(MS, NS, 8, 4, SILU)) return launch_instance<INT_SCALE, MS, NS, 8, 4, SILU>(a, stream);
    }
    return hipErrorInvalidValue;
}
template <bool INT_SCALE, bool SILU, int MS>
hipError_t launch_ns(const FewArgs& a, const FewPlan& p, hipStream_t stream) {
    switch (p.ns) {
        case 1: return launch_waves<INT_SCALE, SILU, MS, 1>(a, p, stream);
        case 2: return launch_waves<INT_SCALE, SILU, MS, 2>(a, p, stream);
        case 3: return launch_waves<INT_SCALE, SILU, MS, 3>(a, p, stream);
        case 4: return launch_waves<INT_SCALE, SILU, MS, 4>(a, p, stream);
        case 5: return launch_waves<INT_SCALE, SILU, MS, 5>(a, p, stream);
        case 6: return launch_waves<INT_SCALE, SILU, MS, 6>(a, p, stream);
        case 7: return launch_waves<INT_SCALE, SILU, MS, 7>(a, p, stream);
        default: return hipErrorInvalidValue;
    }
}
template <bool INT_SCALE, bool SILU>
hipError_t launch_ms(const FewArgs& a, const FewPlan& p, hipStream_t stream) {
    switch (p.ms) {
        case 1: return launch_ns<INT_SCALE, SILU, 1>(a, p, stream);
        case 2: return launch_ns<INT_SCALE, SILU, 2>(a, p, stream);
        case 3: return launch_ns<INT_SCALE, SILU, 3>(a, p, stream);
        case 4: return launch_ns<INT_SCALE, SILU, 4>(a, p, stream);
        default: return hipErrorInvalidValue;
    }
}

template <bool INT_SCALE>
hipError_t launch_grouped(const FewArgs& a, const FewGroups& g, const FewPlan& p, hipStream_t stream) {
    if (p.ms == 4) return p.ns == 2 ? launch_grouped_instance<4, 2, 4, 2, INT_SCALE>(a, g, stream) : launch_grouped_instance<4, 3, 4, 2, INT_SCALE>(a, g, stream);
    switch (p.ns) {
        case 2: return launch_grouped_instance<2, 2, 4, 2, INT_SCALE>(a, g, stream);
        case 3: return launch_grouped_instance<2, 3, 4, 2, INT_SCALE>(a, g, stream);
        case 4: return launch_grouped_instance<2, 4, 4, 2, INT_SCALE>(a, g, stream);
        default: return launch_grouped_instance<2, 5, 4, 2, INT_SCALE>(a, g, stream);
    }
}

// microseconds: a wave's step with its SIMD to itself, a workgroup's start and end (fitted, see few_plan)
double step_us(int ms, int ns) { return 0.062 * ms + 0.025 * ns + 0.014 * ms * ns; }
double ends_us(int ms, int ns) { return 1.1 * (1.0 + 0.11 * ms * ns); }

}  // namespace

// Waves: eight where one workgroup a compute unit is all there is, so that each SIMD still has two (by rows, from the K length on
// where their longer ends are made up for: same tiles, 16 rows and less, K = 12288: 0.71 of four waves' time, K = 4096 0.94, K = 1024
// 1.02; 64 rows 0.97 / 1.03 / 1.05), four otherwise: two workgroups share a unit, one's start and end under the other's loop.
// A ring of four steps for long runs of one or two tiles, where two steps are too little on their way (4096 x 11008, 16 rows: 7.6 -> 7.5 us;
// 3408 x 19328, 8 rows: 12.8 -> 10.4; on short runs the steps that fill up the last turn cost more: 1000 x 1024 3.4 -> 3.7).
// Tiles: a time of both halves of a unit's work, fitted to 359 calls (2 to 64 rows, 1000 to 57344 columns, K 1024 to 28672): on them
// the choice costs 0.8 % on average and 12 % at most.
FewPlan few_plan(int M, int N, int K, bool silu) {
    const int cus = cu_count(), steps = K >> 7, tiles = (N + 15) / 16;
    const int ms = (M + 15) / 16;
    constexpr int kEightFrom[4] = {24, 24, 32, 96};
    FewPlan best{};
    double best_us = 0.0;
    for (int ns = 1; ns <= 7; ++ns) {
        if (!has_instance(ms, ns, 4, 2, silu)) continue;
        const int wgs = (tiles + ns - 1) / ns, per_cu = (wgs + cus - 1) / cus;
        // (two tiles each and nearly every unit taken: four waves with a deeper ring start sooner and read as fast; 8192 x 8192, 16 and
        // 32 rows, 9.6 -> 9.1 and 11.4 -> 10.7 us; 8192 x 28672 27.7 -> 26.9 and 33.5 -> 32.5)
        const bool full = ns == 2 && ms <= 3 && steps >= 64 && 10 * wgs >= 9 * cus;
        const int waves = per_cu == 1 && ns <= 3 && !full && steps >= kEightFrom[ms - 1] ? 8 : 4;
        int run = (steps + waves - 1) / waves;
        const int depth = has_instance(ms, ns, waves, 4, silu) && run >= (ms == 1 ? 8 : 16) ? 4 : 2;  // (K steps)
        run = (run + depth - 1) / depth * depth;
        const double step = step_us(ms, ns), ends = ends_us(ms, ns);
        const double us = waves == 8 ? per_cu * (ends + 2 * run * step) : (per_cu / 2) * (ends + 2 * run * step) + (per_cu % 2) * (ends + run * step);
        if (best.ns == 0 || us < best_us) {
            best = FewPlan{ms, ns, waves, depth, us};
            best_us = us;
        }
    }
    return best;
}

void few_kernel_name(const FewPlan& p, bool int_scale, bool silu, char* buf, size_t len) {
    snprintf(buf, len, "gemm_few_pk_kernel<%d, %d, %d, %d, %s, %s>", p.ms, p.ns, p.waves, p.depth, int_scale ? "true" : "false", silu ? "true" : "false");
}

hipError_t launch_gemm_few_pk(const FewArgs& a, const FewPlan& p, bool int_scale, bool silu, hipStream_t stream) {
    if (silu) return int_scale ? launch_ms<true, true>(a, p, stream) : launch_ms<false, true>(a, p, stream);
    return int_scale ? launch_ms<true, false>(a, p, stream) : launch_ms<false, false>(a, p, stream);
}

hipError_t launch_gemm_few_grouped_pk(const FewArgs& a, const FewGroups& g, const FewPlan& p, bool int_scale, hipStream_t stream) {
    return int_scale ? launch_grouped<true>(a, g, p, stream) : launch_grouped<false>(a, g, p, stream);
}

// The mixture-of-experts form takes the calls of few rows an expert: there the tiled kernel's preparation and its tiles of 256 columns,
// which go through LDS with a barrier a step, cost more than one read of the weights (8 experts, two per token: 28672 x 4096,
// 16 tokens, 115.7 -> 93.0 us, 64 tokens 109 -> 96.7; 4096 x 14336 61.3 -> 47.0 and 63.7 -> 47.9; 4 experts of 6144 x 2048, one per
// token, 32 tokens 18.6 -> 8.6).  At 32 rows an expert the tiled kernel is ahead where the weights are large (28672 x 4096 115.6
// against 123.4 us here) and behind where they are not (4096 x 14336 72.7 and 68.2, 6144 x 2048 23.7 and 10.6).
// Rows are dealt as if the router were uniform (the offsets are on the device): workgroups of 32 rows, of 64 from 24 rows an expert on.
// Within these limits by fitted times of both kernels (408 calls, 1 to 1024 experts, 12 and 18 % off): short K ranges and experts without
// rows, whose workgroups start for nothing, belong to the tiled kernel, whose table leaves them out (128 experts of 15648 x 128, 7 rows, 14.6
// us there and 52 here; 512 of 6192 x 256, 57 rows, 38 and 102; 256 of 8752 x 256, 3524 rows, 128 and 237; 128 of 2048 x 768, 512 rows 33 and
// 36).  With a tenth to spare, on 259 other calls with rows dealt evenly, by Zipf's law, half at one expert or all: 0.52 to 0.61 of the tiled
// kernel's time, two of 1036 slower than there by more than the runs differ (512 experts of 560 x 2432, 12282 rows, by Zipf's law 134 and
// 144 us, all at one 68 and 91).
FewPlan few_grouped_plan(int E, int M, int N, int K) {
    const int tiles = (N + 15) / 16;
    const double rows = (double)M / E;
    if (rows > 40.0 || (rows > 24.0 && (long long)E * tiles > 2048)) return FewPlan{0, 0, 0, 0};
    const int ms = rows <= 10.0 ? 1 : rows <= 24.0 ? 2 : 3;
    const double idle = pow(1.0 - 1.0 / E, M);  // share of the experts that no row comes to
    const double used = E * (1.0 - idle);
    int run = ((K >> 7) + 3) / 4;
    run += run & 1;
    FewPlan best{rows <= 24.0 ? 2 : 4, 0, 4, 2};
    double best_us = 0.0;
    for (int ns = 2; ns <= (best.ms == 2 ? 5 : 3); ++ns) {
        const double per_cu = (tiles + ns - 1) / ns * used / cu_count();
        // rounds of two workgroups a unit, the last one as long as the others
        const double us = per_cu <= 1.05 ? ends_us(ms, ns) + run * step_us(ms, ns) : ceil(per_cu / 2 - 0.05) * (ends_us(ms, ns) + 2 * run * step_us(ms, ns));
        if (best.ns == 0 || us < best_us) {
            best.ns = ns;
            best_us = us;
        }
    }
    const int slots = 2 * cu_count(), wgs = (tiles + best.ns - 1) / best.ns;
    const double bytes = 1e-6 * N * (double)K * used;
    const double here = 3.1 + 0.33 * wgs * E * idle / slots +
                        std::max(1.0, wgs * used / slots) * (1.34 + 0.59 * ends_us(ms, best.ns) + 0.51 * 2 * run * step_us(ms, best.ns)) + 0.075 * bytes;
    const double there = 10.4 + 0.085 * std::max(1.0, (N + 255) / 256 * used / cu_count()) * (19.5 + (K >> 7)) + 0.112 * bytes;
    return here < 0.9 * there ? best : FewPlan{0, 0, 0, 0};
}

void few_grouped_kernel_name(const FewPlan& p, bool int_scale, char* buf, size_t len) {
    snprintf(buf, len, "gemm_few_grouped_pk_kernel<%d, %d, %d, %d, %s>", p.ms, p.ns, p.waves, p.depth, int_scale ? "true" : "false");
}

// Moderate numbers of rows in tiles of 48 or 64: the plan and its time in microseconds, launch and weights' way from memory included (the
// fit of few_plan; 65 x 4096 x 4096 8.2 by it and 8.8 measured, 300 x 6144 x 4096 15.7 and 16.8, 512 x 12288 x 4096 41.7 and 40.8, 300 x
// 28672 x 4096 66 and 60).
FewPlan rows_plan(int M, int N, int K, bool silu, double* us_out) {
    const int cus = cu_count();
    int run = ((K >> 7) + 3) / 4;
    run += run & 1;
    FewPlan best{0, 0, 4, 2};
    double best_us = 0.0;
    for (int ms = 3; ms <= 4; ++ms)
        for (int ns = 3; ns <= (ms == 3 ? 5 : 4); ++ns) {
            if (silu && ns % 2 != 0) continue;
            const long long wgs = (long long)((N + 16 * ns - 1) / (16 * ns)) * ((M + 16 * ms - 1) / (16 * ms));
            const long long per_cu = (wgs + cus - 1) / cus;
            const double step = step_us(ms, ns), ends = ends_us(ms, ns);
            const double us = (double)(per_cu / 2) * (ends + 2 * run * step) + (double)(per_cu % 2) * (ends + run * step);
            if (best.ns == 0 || us < best_us) {
                best.ms = ms;
                best.ns = ns;
                best_us = us;
            }
        }
    *us_out = 1.9 + best_us + 0.064e-6 * N * (double)K;
    return best;
}

void rows_kernel_name(const FewPlan& p, bool silu, char* buf, size_t len) {
    snprintf(buf, len, "gemm_rows_pk_kernel<%d, %d, %d, %d, %s>", p.ms, p.ns, p.waves, p.depth, silu ? "true" : "false");
}

hipError_t launch_gemm_rows_pk(const FewArgs& a, const FewPlan& p, bool silu, hipStream_t stream) {
    if (silu) return p.ms == 3 ? launch_rows_instance<3, 4, true>(a, stream) : launch_rows_instance<4, 4, true>(a, stream);
    if (p.ms == 4) return p.ns == 3 ? launch_rows_instance<4, 3, false>(a, stream) : launch_rows_instance<4, 4, false>(a, stream);
    if (p.ns == 3) return launch_rows_instance<3, 3, false>(a, stream);
    return p.ns == 4 ? launch_rows_instance<3, 4, false>(a, stream) : launch_rows_instance<3, 5, false>(a, stream);
}

}  // namespace intscale
