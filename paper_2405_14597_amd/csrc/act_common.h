// Device helpers shared by the activation quantiser and by the kernels that fold it into the operator producing the
// activation: wave and workgroup reductions, and Appendix A.1's code for eight fp16 values at a time.  The quotient
// x / s is a true IEEE fp32 division and rounding is round-half-to-even, because they decide the integer code.
#pragma once
#include "is_common.h"

namespace intscale {

// Maximum over the 64 lanes of a wave, for values that are >= 0 in every lane (an absmax): their bit patterns order
// like unsigned integers.  Four lane-swizzled steps inside each row of 16 lanes (neighbour, pair, mirrored half,
// mirrored row), then the four row results meet in scalar registers.  No trip through the LDS crossbar, whose
// latency would sit six times in a row on the critical path of a one-token kernel.
__device__ __forceinline__ float wave_max(float v) {
    unsigned x = __float_as_uint(v);
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true));   // quad_perm [1,0,3,2]
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, true));   // quad_perm [2,3,0,1]
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, true));  // row_half_mirror
    x = max(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, true));  // row_mirror
    const unsigned r0 = __builtin_amdgcn_readlane((int)x, 0), r1 = __builtin_amdgcn_readlane((int)x, 16);
    const unsigned r2 = __builtin_amdgcn_readlane((int)x, 32), r3 = __builtin_amdgcn_readlane((int)x, 48);
    return __uint_as_float(max(max(r0, r1), max(r2, r3)));
}

// Largest magnitude of eight fp16 values, 0 if none of them is a number.  Magnitudes order like unsigned integers, so the maxima
// are taken on their bits, two values an instruction (11 instructions with the test below and the caller's running maximum, where
// converting first takes 18).  A NaN, signalling ones among them, is then the largest: where a wave meets one, its maxima are taken again in
// floating point, where a NaN loses against a number.
__device__ __forceinline__ float absmax8(uint4 v) {
    auto larger = [](uint32_t a, uint32_t b) {
        uint32_t r;
        asm("v_pk_max_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
        return r;
    };
    constexpr uint32_t kAbs = 0x7FFF7FFFu, kInf = 0x7C00u;
    const uint32_t m2 = larger(larger(v.x & kAbs, v.y & kAbs), larger(v.z & kAbs, v.w & kAbs));
    const uint32_t m = max(m2 & 0xFFFFu, m2 >> 16);
    float r = __half2float(__ushort_as_half((unsigned short)m));
    if (__builtin_expect(__any(m > kInf), 0)) {
        const __half2* h = reinterpret_cast<const __half2*>(&v);
        r = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float2 f = __half22float2(h[i]);
            r = fmaxf(r, fmaxf(fabsf(f.x), fabsf(f.y)));
        }
    }
    return r;
}

// e^t and SiLU(g) * u as fixed sequences of separately rounded single-precision operations (no contraction into
// fused multiply-adds): the fp16 result may decide integer codes further on, so every user computes it the same way.
// Shorter forms stand in where they give the same bits.  n = rint(t log2 e) is read off the sum with 2^23 + 2^22, whose low
// bits are also the exponent that 2^n adds to p (|n| <= 127 and p lies in [0.7, 1.5], so the result stays normal);
// n * ln2_hi is exact, so subtracting it in a fused multiply-add rounds once all the same.
// The definition clamps t at 88, this at 87: above it SiLU is about -1e-36 either way (its product with any finite fp16 value is
// a zero of the same sign), and 1 + e^t stays below 2^126, where the reciprocal that silu_mul takes is a normal number.  A
// smaller one is flushed to 0, and 0 times an infinite up value is no infinity.
constexpr float kExpMax = 87.0f;

__device__ __forceinline__ float exp_steps(float t) {
#pragma clang fp contract(off)
    constexpr float kRound = 12582912.0f;
    t = fminf(fmaxf(t, -87.0f), kExpMax);
    const float shifted = fmaf(t, 1.4426950408889634f, kRound);
    const float n = shifted - kRound;
    const float r = fmaf(-n, 0.693145751953125f, t) - n * 1.428606765330187e-06f;
    float p = (float)(1.0 / 720.0);
    p = p * r + (float)(1.0 / 120.0);
    p = p * r + (float)(1.0 / 24.0);
    p = p * r + (float)(1.0 / 6.0);
    p = p * r + 0.5f;
    p = p * r + 1.0f;
    p = p * r + 1.0f;
    return __uint_as_float(__float_as_uint(p) + (__float_as_uint(shifted) << 23));
}

// A single-precision value that is about to be converted to fp16, as the rounded fp32 value it is: without this the
// compiler may merge the last multiply into the conversion (v_fma_mixlo_f16 rounds the exact product once, straight to
// fp16), which differs from "round to fp32, then to fp16" wherever the fp32 result falls on an fp16 tie.
__device__ __forceinline__ float rounded_f32(float v) {
    asm("" : "+v"(v));
    return v;
}

// g holds an fp16 value, so SiLU(g) takes one of 2^16 values, and the short form of the division below (reciprocal, one
// correction of the quotient, the fix-up for infinities and NaN) has been compared with the true division on every one of
// them: the same bits wherever the quotient is above 1e-30, and the same sign below that, where it is no zero and its product with
// a finite fp16 value rounds to one.  6 instructions where the general division takes 11; with the shorter e^t above 32 instead of
// 41 per element, SiLU * up and quantiser at 2048 x 28672: 85 -> 64 us (4.6 TB/s; with the
// row spread over 1024 lanes, see the launcher).
__device__ __forceinline__ float silu_mul(float g, float u) {
#pragma clang fp contract(off)
    const float d = 1.0f + exp_steps(-g);
    const float y = __builtin_amdgcn_rcpf(d);
    float q = g * y;
    q = fmaf(fmaf(-d, q, g), y, q);
    q = __builtin_amdgcn_div_fixupf(q, d, g);
    return rounded_f32(q * u);
}

__device__ __forceinline__ int quant_code(float x, float s, float lo, float hi) {
    // s > 0 is checked by the caller
    float r = rintf(x / s);
    r = fminf(fmaxf(r, lo), hi);
    return (int)r;
}

// ---------------------------------------------------------------------------------------------------------
// Activations: one workgroup per token row.  Pass 1 finds the row's absmax (16-byte loads), pass 2 re-reads the
// row (it is at most a few tens of KB, so it comes back from L2) and writes 8 codes per lane as one 8-byte store.
// ---------------------------------------------------------------------------------------------------------
constexpr int kActThreads = 256;

// Appendix A.1 codes of eight values of one token row, rne(x / s) with the quotient rounded as a true division rounds it.
// A division costs a dozen instructions, so the codes are first read off products with two neighbours of 1 / s: with
// r = fl(1 / s), the exact products x * r (1 - 2^-21) and x * r (1 + 2^-21) lie on either side of both x / s and its fp32
// rounding (r, its neighbours and the quotient are off by at most a few 2^-24 of their size), and rounding to an integer is
// monotone, so where the two agree the quotient rounds to the same integer.  Where they differ anywhere in a wave (at
// |x / s| <= 127 about one chunk of 512 values in fifty) all its values are redone with the division itself.
// One fused multiply-add per product does everything: added to 2^23 + 2^22 + an offset the exact product is rounded to an integer,
// ties to even, and the sum's lowest byte is the code + the offset.  The fp16 operand is converted inside the instruction
// (v_fma_mix_f32), the comparison is one or-of-xor per value, the packing three byte permutes per four codes: 4 instructions a
// value where multiply, round, distance, running maximum, offset and saturating conversion took 7.  Stand-alone quantiser,
// 4096 x 14336: 31.0 -> 29.6 us (5.9 TB/s: bound by memory now); quantising preparation of the tiled kernel, 4096 x 4096: 22.8
// -> 20.3 us.
constexpr float kCodeMagic = 12582912.0f;  // + the offset

__device__ __forceinline__ uint32_t low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
    const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0C0C0400u), cd = __builtin_amdgcn_perm(d, c, 0x0C0C0400u);
    return __builtin_amdgcn_perm(cd, ab, 0x05040100u);
}

// Values as offset_codes wants them: all zero where there is no scale, i.e. where every number of the row or group is zero (a
// NaN among them has code 0 as well, but times a reciprocal of 0 it is no 0).
__device__ __forceinline__ uint4 zero_without_scale(uint4 v, float s) {
    if (__builtin_expect(__any(!(s > 0.0f)), 0)) v = s > 0.0f ? v : make_uint4(0u, 0u, 0u, 0u);
    return v;
}

// N values' codes + OFFSET in the low bytes of c[] (beside a scale a value that is no number gives byte 0, the lowest code, as the
// clamp of a NaN does)
template <int OFFSET, int N>
__device__ __forceinline__ void offset_codes(const float (&x)[N], float s, uint32_t (&c)[N]) {
    const float r = s > 0.0f ? 1.0f / s : 0.0f;
    const float r_lo = r * (1.0f - 0x1p-21f), r_hi = r * (1.0f + 0x1p-21f);
    uint32_t apart = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        c[i] = __float_as_uint(fmaf(x[i], r_lo, kCodeMagic + OFFSET));
        const uint32_t other = __float_as_uint(fmaf(x[i], r_hi, kCodeMagic + OFFSET));
        // apart |= c[i] ^ other, in one instruction (written out in C it becomes a flag per value and the flags are packed)
        asm("v_bitop3_b32 %0, %1, %2, %0 bitop3:0xbe" : "+v"(apart) : "v"(c[i]), "v"(other));
    }
    if (__builtin_expect(__any(apart != 0), 0)) {
        const float by = s > 0.0f ? s : 1.0f;
#pragma unroll
        for (int i = 0; i < N; ++i) c[i] = __float_as_uint(rintf(x[i] / by) + (kCodeMagic + OFFSET));
    }
}

__device__ __forceinline__ uint2 quantize8(uint4 v, float s) {
    v = zero_without_scale(v, s);
    const __half2* h = reinterpret_cast<const __half2*>(&v);
    float x[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float2 f = __half22float2(h[i]);
        x[2 * i] = f.x;
        x[2 * i + 1] = f.y;
    }
    uint32_t c[8];
    offset_codes<128>(x, s, c);  // (flipping the top bit of a byte turns code + 128 into two's complement)
    return make_uint2(low_bytes(c[0], c[1], c[2], c[3]) ^ 0x80808080u, low_bytes(c[4], c[5], c[6], c[7]) ^ 0x80808080u);
}

// NW = waves in the workgroup; `red` holds NW floats
template <int NW = kActThreads / kWave>
__device__ __forceinline__ float block_max(float v, float* red) {
    v = wave_max(v);
    if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) v = fmaxf(v, red[i]);
    return v;
}

}  // namespace intscale
