// Device helpers shared by the activation kernels: bf16 unpacking and rounding, maxima over neighbouring lanes, and
// the INT4 quantizer of one token's eight channels in the GEMM's 6-bit operand form
// (arXiv 2411.05007 Eq. 1 per group of 64; App. "Implementation Details").
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout.h"

namespace svdq {

__device__ __forceinline__ float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
// round-to-nearest-even fp32 -> bf16 of two values (v_cvt_pk_bf16_f32), lo in the low half
__device__ __forceinline__ uint32_t bf16_rne_pair(float lo, float hi) {
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    bf16x2_t v;
    v[0] = (__bf16)lo;
    v[1] = (__bf16)hi;
    return __builtin_bit_cast(uint32_t, v);
}

// maximum over the 4 lanes of a quad
__device__ __forceinline__ float max_over_4_lanes(float a) {
    a = fmaxf(a, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), 0xB1, 0xf, 0xf, true)));    // quad_perm [1,0,3,2]
    a = fmaxf(a, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), 0x4E, 0xf, 0xf, true)));    // quad_perm [2,3,0,1]
    return a;
}
// maximum over the 8 lanes l % 8 = 0..7
__device__ __forceinline__ float max_over_8_lanes(float a) {
    a = max_over_4_lanes(a);
    a = fmaxf(a, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, a), 0x141, 0xf, 0xf, true)));   // row_half_mirror
    return a;
}

// Eq. 1 for a token's group of 64 with the maximum `amax`: s = max|x| / q_max, stored as fp16 (`sbits`); returns 1 / s, the factor
// that turns x^ into its code (0 for a group of zeros).  w4_group_rcp: a lane holds 8 channels of the group, the other 56 sit in the
// 7 lanes beside it.
__device__ __forceinline__ float w4_rcp_of(float amax, uint32_t &sbits) {
    // amax / 7.0f and 1.0f / s, both correctly rounded like the IEEE divisions they stand for, in three instructions
    // each: a product with the rounded reciprocal (1/7 as a constant, v_rcp_f32 for s, good to one ulp), the exact
    // remainder by FMA, one correction by FMA.  For the division by 7 this equals the IEEE quotient for every finite
    // fp32 numerator, and for 1/s for every positive fp16 s even from a start two ulps off (both checked exhaustively
    // on the host).
    constexpr float kInv7 = 0x1.24924ap-3f;                  // 1.0f / 7.0f
    const float q0 = amax * kInv7;
    float s32 = __builtin_fmaf(__builtin_fmaf(-7.0f, q0, amax), kInv7, q0);
    s32 = fminf(s32, 65504.0f);
    const _Float16 sh = (_Float16)s32;
    const float sc = (float)sh;
    const float den = sc > 0.f ? sc : 1.0f;                  // branch-free: the reciprocal always runs
    const float y0 = __builtin_amdgcn_rcpf(den);
    const float rcp_any = __builtin_fmaf(__builtin_fmaf(-den, y0, 1.0f), y0, y0);
    sbits = __builtin_bit_cast(uint16_t, sh);
    return sc > 0.f ? rcp_any : 0.f;
}
__device__ __forceinline__ float w4_group_rcp(const float (&xh)[8], uint32_t &sbits) {
    float amax = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(xh[e]));
    return w4_rcp_of(max_over_8_lanes(amax), sbits);
}

// The codes of up to four such 8-channel runs at once, in the operand form of the GEMM's matrix instruction
// (layout.h): 6 bits per code - sign, two zero bits, magnitude - i.e. the 6-bit float (E2M3) of value q / 8, which is
// what v_cvt_scalef32_2xpk16_fp6_f32 makes of x^ / s with the scale operand 8: it divides by 8 and rounds to the
// nearest multiple of 1/8, ties to even, exactly the rounding of Eq. 1 for |x^ / s| < 7.5; the clamp to +-7 before it
// stands for the clip of Eq. 1 (it acts only where s was rounded down hard, next to the bottom of the fp16 range, or
// cut off at its top).  The instruction takes two vectors of 16 and interleaves them: element i of the first lands in
// field 2 i, of the second in field 2 i + 1; so run j (j = 0..3) gives its even channels to elements 4 j .. 4 j + 3 of
// the first vector and its odd channels to those of the second, and its 8 codes come out as bits 48 j .. 48 j + 47
// of the 192, channel e at bit 6 e of the run.  A zero code keeps the sign of x^, which the format ignores.
typedef float act_floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t act_u32x6 __attribute__((ext_vector_type(6)));
template <int RUNS>
__device__ __forceinline__ act_u32x6 w4_codes(const float (*const (&xh)[RUNS])[8], const float (&rcp)[RUNS]) {
    act_floatx16 ev, od;
#pragma unroll
    for (int i = 0; i < 16; ++i) ev[i] = od[i] = 0.f;
#pragma unroll
    for (int j = 0; j < RUNS; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ev[4 * j + i] = __builtin_amdgcn_fmed3f((*xh[j])[2 * i] * rcp[j], -7.0f, 7.0f);
            od[4 * j + i] = __builtin_amdgcn_fmed3f((*xh[j])[2 * i + 1] * rcp[j], -7.0f, 7.0f);
        }
    return __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(ev, od, 8.0f);
}
// the codes of 32 neighbouring channels that one lane holds: a lane's operand registers as they are
__device__ __forceinline__ act_u32x6 w4_codes32(const float (&xh)[32], float rcp) {
    act_floatx16 ev, od;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        ev[i] = __builtin_amdgcn_fmed3f(xh[2 * i] * rcp, -7.0f, 7.0f);
        od[i] = __builtin_amdgcn_fmed3f(xh[2 * i + 1] * rcp, -7.0f, 7.0f);
    }
    return __builtin_amdgcn_cvt_scalef32_2xpk16_fp6_f32(ev, od, 8.0f);
}
// run j of such a result as the 48 bits (lo: bits 0-31, hi: bits 32-47) that one lane stores
__device__ __forceinline__ void w4_run48(const act_u32x6 &r, int j, uint32_t &lo, uint32_t &hi) {
    const int w = (3 * j) >> 1;
    if (j & 1) {
        lo = (r[w] >> 16) | (r[w + 1] << 16);
        hi = r[w + 1] >> 16;
    } else {
        lo = r[w];
        hi = r[w + 1] & 0xffffu;
    }
}


// Where the codes and scales of a wavefront's 16 tokens of one group meet in LDS, in the byte order of the activation block
// (kActOutStage bytes in three runs: the two k-halves and the scales), and how they leave.  Lane 8 r8 + c8 holds channels
// 8 c8 .. + 7 of tokens r8 and r8 + 8: half of one 16-channel triple (three registers of the GEMM's 6-bit operand form,
// layout.h).  The even lane of a pair stores the triple's first two dwords, the odd lane the third, and then lane c8 = 1
// the token's scale dword, the other odd lanes the third dword once more (same value to the same address).
struct W4Stage {
    int a, b, a2, b2, c8;
    __device__ __forceinline__ W4Stage(int r8, int c8_) : c8(c8_) {
        a = 384 * (c8 >> 2) + 24 * r8 + 12 * ((c8 & 3) >> 1) + ((c8 & 1) ? 8 : 0);
        b = a + 24 * 8;
        a2 = (c8 & 1) ? (c8 == 1 ? 768 + 4 * r8 : a) : a + 4;
        b2 = (c8 & 1) ? (c8 == 1 ? 768 + 4 * (r8 + 8) : b) : b + 4;
    }
    // the 48 bits of codes and the scale of token r8 (alo, ahi, sa) and of token r8 + 8 as the words that go to a, b, a2, b2
    __device__ __forceinline__ void words(uint32_t alo, uint32_t ahi, uint32_t sa, uint32_t blo, uint32_t bhi, uint32_t sb, uint32_t &a1, uint32_t &b1, uint32_t &a2v,
                                          uint32_t &b2v) const {
        // Two neighbouring lanes hold the 16 codes of one triple = 96 bits: dword 0 is the even lane's low word,
        // dword 1 the even lane's high 16 bits and the odd lane's low 16, dword 2 the rest of the odd lane.
        const uint32_t na = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)alo, 0xB1, 0xf, 0xf, true);      // the pair's other lane
        const uint32_t nb = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)blo, 0xB1, 0xf, 0xf, true);
        const bool odd = c8 & 1;
        a1 = odd ? ((alo >> 16) | (ahi << 16)) : alo;                // first store: dword 2 (odd) or dword 0 (even)
        b1 = odd ? ((blo >> 16) | (bhi << 16)) : blo;
        a2v = odd ? (c8 == 1 ? sa : a1) : (ahi | (na << 16));        // second: the scale, dword 2 again, or dword 1
        b2v = odd ? (c8 == 1 ? sb : b1) : (bhi | (nb << 16));
    }
    __device__ __forceinline__ void put(unsigned char *stage, uint32_t alo, uint32_t ahi, uint32_t sa, uint32_t blo, uint32_t bhi, uint32_t sb) const {
        // (all four words are made before the first is stored: made in between the stores, the second two cost the ranks
        // above 64 four registers and, with a long K, 1 us of a launch: M = 4608, K = 12288, rank 128 71.2 against 69.9)
        uint32_t a1, b1, a2v, b2v;
        words(alo, ahi, sa, blo, bhi, sb, a1, b1, a2v, b2v);
        *reinterpret_cast<uint32_t *>(stage + a) = a1;
        *reinterpret_cast<uint32_t *>(stage + b) = b1;
        *reinterpret_cast<uint32_t *>(stage + a2) = a2v;
        *reinterpret_cast<uint32_t *>(stage + b2) = b2v;
    }
    // eight tokens: the first eight rows of each run
    __device__ __forceinline__ void put(unsigned char *stage, uint32_t alo, uint32_t ahi, uint32_t sa) const {
        uint32_t a1, b1, a2v, b2v;
        words(alo, ahi, sa, 0u, 0u, 0u, a1, b1, a2v, b2v);
        *reinterpret_cast<uint32_t *>(stage + a) = a1;
        *reinterpret_cast<uint32_t *>(stage + a2) = a2v;
    }
};
// where lane l's 16 bytes of such a stage belong in the group's activation blocks (lanes below kActOutStage / 16)
__device__ __forceinline__ int w4_stage_out(int m0, int lane) {
    const int half16 = (m0 >> 4) & 1;
    return (m0 / 32) * kW4ABlock + (lane < 24 ? 384 * half16 + 16 * lane : lane < 48 ? 768 + 384 * half16 + 16 * (lane - 24) : kW4ACodes + 64 * half16 + 16 * (lane - 48));
}
// and of a stage of eight tokens: lanes 0-11 and 12-23 the k-halves, 24 and 25 the scales
__device__ __forceinline__ int w4_stage_out8(int m0, int lane) {
    const int half16 = (m0 >> 4) & 1, half8 = (m0 >> 3) & 1;
    return (m0 / 32) * kW4ABlock + (lane < 12 ? 384 * half16 + 192 * half8 + 16 * lane
                                    : lane < 24 ? 768 + 384 * half16 + 192 * half8 + 16 * (lane - 12)
                                                : kW4ACodes + 64 * half16 + 32 * half8 + 16 * (lane - 24));
}

// Eq. 1 for one MXFP4 block (the 32 channels held by 4 neighbouring lanes): the scale is the smallest power
// of two s = 2^e >= 2^-126 with max|x| <= 6 s, found from the exponent and mantissa bits of the maximum
// (max|x| = 1.m * 2^(E - 127) <= 1.5 * 2^(e + 2)  <=>  e = E - 129, one more if 1.m > 1.5), stored as the
// byte e + 127 (0 for an all-zero block); the codes come from the hardware conversion, which divides by
// the scale's power of two and rounds to the nearest E2M1 element, ties to even, saturating.
__device__ __forceinline__ float fp4_scale_of(float amax, uint32_t &sbyte) {
    const uint32_t bits = __float_as_uint(amax);
    int byte = (int)(bits >> 23) - 2 + ((bits & 0x7fffffu) > 0x400000u ? 1 : 0);
    byte = byte < 1 ? 1 : (byte > 254 ? 254 : byte);
    const bool zero = !(amax > 0.f);
    sbyte = zero ? 0u : (uint32_t)byte;
    return __uint_as_float((zero ? 127u : (uint32_t)byte) << 23);
}
__device__ __forceinline__ uint32_t fp4_word(float a, float b, float c, float d, float e, float f, float g, float h, float scale) {
    uint32_t w = 0u;
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, a, b, scale, 0);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, c, d, scale, 1);
    w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, e, f, scale, 2);
    return __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, g, h, scale, 3);
}
// a lane holds 8 channels of the block, the other 24 sit in the rest of its quad
__device__ __forceinline__ void fp4_encode(const float (&xh)[8], uint32_t &word, uint32_t &sbyte) {
    float amax = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(xh[e]));
    const float scale = fp4_scale_of(max_over_4_lanes(amax), sbyte);
    word = fp4_word(xh[0], xh[1], xh[2], xh[3], xh[4], xh[5], xh[6], xh[7], scale);
}
// a lane holds the whole block, `amax` its maximum
__device__ __forceinline__ uint4 fp4_encode32(const float (&xh)[32], float amax, uint32_t &sbyte) {
    const float scale = fp4_scale_of(amax, sbyte);
    auto word = [&](int e) { return fp4_word(xh[e], xh[e + 1], xh[e + 2], xh[e + 3], xh[e + 4], xh[e + 5], xh[e + 6], xh[e + 7], scale); };
    return make_uint4(word(0), word(8), word(16), word(24));
}

// Partial H [runs][Mpad][rank] in place of H: how a launch says so in H's first 16 bytes, and how a reader of H follows it.
__device__ __forceinline__ void h_in_parts(float *H, const float *hpart, int runs) {
    *reinterpret_cast<uint4 *>(H) = make_uint4(kHInParts0, kHInParts1, (uint32_t)runs, (uint32_t)((hpart - H) / 64));
}
__device__ __forceinline__ float h_element(const float *H, size_t idx, int Mpad, int rank) {
    const uint4 w = *reinterpret_cast<const uint4 *>(H);
    if (w.x != kHInParts0 || w.y != kHInParts1) return H[idx];
    const float *part = H + (size_t)w.w * 64 + idx;
    float h = 0.f;
    for (uint32_t r = 0; r < w.z; ++r) h += part[(size_t)r * Mpad * rank];
    return h;
}

}  // namespace svdq
