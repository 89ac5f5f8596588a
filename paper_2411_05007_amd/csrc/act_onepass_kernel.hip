// Activation kernel in one pass (arXiv 2411.05007 Sec. 4.3, Fig. 6b): smoothing, quantization (Eq. 1) and the down projection
// H = X L1s, a workgroup of sixteen wavefronts to 16 or 8 tokens and all of their K.  Wavefront w has groups w, w + 16, ..., up to NG
// of them, requested up to six at a time, long before they are used; nothing is parked or added up across workgroups, and
// there is one barrier.
//   FMT 0, 1 (INT4, MXFP4): groups are independent; what act_kernel.hip does, with more requests in flight per CU.
//   FMT 2 (INT8, one scale per token; App. "Implementation Details"): a token's scale needs its maximum over all of K before
//   the first code can be written, so the workgroup holds its tokens in registers from the one read to the codes.
// Bound: one CU's rate of small requests, X and the L1 fragments that every workgroup reads (M = 4096, K = 4608, rank 32, INT4:
// 16 us against 18 of act_kernel.hip, 38 MB of X), and where the workgroups are fewer than the CUs by the time of one of them
// (INT8, M = 1337, K = 3072, 16 tokens: vector instructions for a third of it, the rest waiting): eight tokens halve its loads of X, its
// vector instructions and its stores.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "act_common.h"
#include "buffer.h"
#include "kernels.h"
#include "layout.h"
#include "lds_limit.h"

namespace svdq {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr int kWaves = 16;

// LDS: the tokens' maxima per wavefront, then one block per wavefront: X of one group on its way from the load map to the
// operand map (rows padded to 144 bytes), at the end the wavefront's partial H
template <int RB>
struct OnePassLds {
    static constexpr int kXRow = 144, kRedRow = RB * 16 + 1;
    static constexpr int kBlock = 16 * kXRow > 16 * kRedRow * 4 ? 16 * kXRow : (16 * kRedRow * 4 + 15) / 16 * 16;
    static constexpr int kMax = kWaves * 16 * 4;
    static constexpr int kWave = kBlock + kActOutStage;                  // and the staging block of the INT4 codes
    static constexpr int kBytes = kMax + kWaves * kWave;
};

// RB: column blocks of 16 of the projection (0: none); NG: groups a wavefront holds; TOK: tokens of a workgroup, 16 or 8
template <int FMT, int RB, int NG, int TOK>
__global__ __launch_bounds__(kWaves * 64, 1) void act_onepass_kernel(ActParams p) {
    using L = OnePassLds<RB>;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, blk = lane >> 4;      // MFMA operand / accumulator map
    constexpr bool kTwo = TOK == 16;
    const int r8 = lane >> 3, c8 = lane & 7;         // load map: tokens r8 and (of sixteen) r8 + 8, channels 8 c8 .. + 7 of a group
    const int m0 = blockIdx.x * TOK, ma = m0 + r8, mb = ma + 8;
    const int rb = p.rank / 16;

    // rows past M read the last row; what they produce lands in padding rows and is never used
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.X, (size_t)p.M * p.K * 2);
    const __amdgpu_buffer_rsrc_t rs_r = make_rsrc(p.rinv, (size_t)p.K * 4);
    const __amdgpu_buffer_rsrc_t rs_l = make_rsrc(p.l1s, (size_t)p.K * p.rank * 2);
    const __amdgpu_buffer_rsrc_t rs_c = make_rsrc(p.codes, FMT == 2 ? (size_t)p.K * p.Mpad : FMT == 1 ? (size_t)p.G * p.Mpad * kFp4RowBytes : w4_a_bytes(p.G, p.Mpad));
    const __amdgpu_buffer_rsrc_t rs_s = make_rsrc(p.sx, FMT == 1 ? fp4_scale_bytes(p.G, p.Mpad) : 0);
    // (byte offsets below 2^32: the entry point refuses batches of 2^31 elements or more; unsigned on purpose)
    const int vxa = (int)(((uint32_t)(ma < p.M ? ma : p.M - 1) * (uint32_t)p.K + 8u * (uint32_t)c8) * 2u);
    const int vxb = (int)(((uint32_t)(mb < p.M ? mb : p.M - 1) * (uint32_t)p.K + 8u * (uint32_t)c8) * 2u);
    const int vca = FMT == 2 ? (int)i8_code_offset(8 * c8, p.Mpad, ma) : (int)fp4_code_offset(0, p.Mpad, ma, c8 >> 2) + 4 * (c8 & 3);
    const int vcb = FMT == 2 ? (int)i8_code_offset(8 * c8, p.Mpad, mb) : (int)fp4_code_offset(0, p.Mpad, mb, c8 >> 2) + 4 * (c8 & 3);
    const int vsx = (int)fp4_scale_offset(0, p.Mpad, kTwo && (c8 & 1) ? mb : ma, c8 >> 2);
    const W4Stage w4(r8, c8);
    const int vout = kTwo ? w4_stage_out(m0, lane) : w4_stage_out8(m0, lane);
    // (of eight tokens, the staging block's three runs are filled by half)
    const int vstage = kTwo ? 16 * lane : lane < 12 ? 16 * lane : lane < 24 ? 384 + 16 * (lane - 12) : 768 + 16 * (lane - 24);
    constexpr int kStageLanes = kTwo ? kActOutStage / 16 : 26;
    auto group = [&](int i) { return wave + kWaves * i; };
    auto load_b128 = [&](__amdgpu_buffer_rsrc_t rs, int v, int s, bool nt) {
        return __builtin_bit_cast(uint4, nt ? __builtin_amdgcn_raw_buffer_load_b128(rs, v, s, 2) : __builtin_amdgcn_raw_buffer_load_b128(rs, v, s, 0));
    };

    // everything that does not depend on anything is requested at once (a group past K: nothing, zeros)
    constexpr int kX = FMT == 2 || NG < 3 ? NG : 3;
    uint4 xa[kX], xb[kX];
    auto load_x = [&](int i) {
        xa[i % kX] = xb[i % kX] = make_uint4(0u, 0u, 0u, 0u);
        if (group(i) < p.G) {
            xa[i % kX] = load_b128(rs_x, vxa, group(i) * 128, true);
            if (kTwo) xb[i % kX] = load_b128(rs_x, vxb, group(i) * 128, true);
        }
    };
    float4 r0[NG], r1[NG];
    // INT8: x^ stays in registers from the maximum to the codes, or X does, and 1 / lambda is loaded again
    constexpr bool kKeep = FMT == 2 && NG * (TOK / 8) <= 6;
    float keep[kKeep ? NG : 1][TOK / 8][8];
#pragma unroll
    for (int i = 0; i < kX; ++i) load_x(i);
    __builtin_amdgcn_sched_barrier(0);
    int vr = 32 * c8;
    auto load_rinv = [&](int i) {
        r0[i] = __builtin_bit_cast(float4, load_b128(rs_r, vr, group(i) < p.G ? group(i) * 256 : 0, false));
        r1[i] = __builtin_bit_cast(float4, load_b128(rs_r, vr + 16, group(i) < p.G ? group(i) * 256 : 0, false));
    };
    struct Frags { uint4 b[RB > 0 ? 2 * RB : 1]; };
    auto load_l1 = [&](int i) {
        Frags f;
        const int sg = (group(i) < p.G ? group(i) : 0) * 2 * rb * 1024;
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            const int cc = c < rb ? c : rb - 1;      // blocks past the rank repeat the last one; their sums are dropped
            f.b[2 * c] = load_b128(rs_l, lane * 16, sg + cc * 1024, false);
            f.b[2 * c + 1] = load_b128(rs_l, lane * 16, sg + (rb + cc) * 1024, false);
        }
        return f;
    };
#pragma unroll
    for (int i = 0; i < (kKeep && NG <= 3 ? NG : 2); ++i) load_rinv(i);
    Frags fr = load_l1(0);
    __builtin_amdgcn_sched_barrier(0);

    auto smooth = [&](uint4 x, const float4 &s0, const float4 &s1, float (&o)[8]) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
        const float r[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            o[2 * e] = bf16lo(w[e]) * r[2 * e];
            o[2 * e + 1] = bf16hi(w[e]) * r[2 * e + 1];
        }
    };
    unsigned char *block = lds + L::kMax + wave * L::kWave;
    floatx4 acc[RB > 0 ? RB : 1];
#pragma unroll
    for (int c = 0; c < (RB > 0 ? RB : 1); ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
    float amax_a = 0.f, amax_b = 0.f;
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        float ta[8], tb[8];
        smooth(xa[i % kX], r0[i], r1[i], ta);
        if (kTwo) smooth(xb[i % kX], r0[i], r1[i], tb);
        if (!(kKeep && NG <= 3)) {
            __builtin_amdgcn_sched_barrier(0);
            if (i + 2 < NG) load_rinv(i + 2);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (FMT == 2) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                amax_a = fmaxf(amax_a, fabsf(ta[e]));
                if (kTwo) amax_b = fmaxf(amax_b, fabsf(tb[e]));
                if (kKeep) {
                    keep[kKeep ? i : 0][0][e] = ta[e];
                    if (kTwo) keep[kKeep ? i : 0][TOK / 8 - 1][e] = tb[e];
                }
            }
        } else if (group(i) < p.G) {
            if constexpr (FMT == 1) {
                uint32_t wa, wb, ba, bb;
                fp4_encode(ta, wa, ba);
                if (kTwo) fp4_encode(tb, wb, bb);
                // the four lanes of a block write the same scale byte (of sixteen tokens, an even c8 that of token r8, an odd one that of r8 + 8)
                const int sc = group(i) * p.Mpad * kFp4RowBytes;
                __builtin_amdgcn_raw_buffer_store_b32(wa, rs_c, vca, sc, 0);
                if (kTwo) __builtin_amdgcn_raw_buffer_store_b32(wb, rs_c, vcb, sc, 0);
                __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(kTwo && (c8 & 1) ? bb : ba), rs_s, vsx, (group(i) >> 2) * p.Mpad * 8 + (group(i) & 3), 0);
            } else {
                unsigned char *stage = block + L::kBlock;
                if constexpr (kTwo) {
                    uint32_t sa, sb, alo, ahi, blo, bhi;
                    const float rcp[2] = {w4_group_rcp(ta, sa), w4_group_rcp(tb, sb)};
                    const float(*const runs[2])[8] = {&ta, &tb};
                    const act_u32x6 q = w4_codes<2>(runs, rcp);
                    w4_run48(q, 0, alo, ahi);
                    w4_run48(q, 1, blo, bhi);
                    w4.put(stage, alo, ahi, sa, blo, bhi, sb);
                } else {
                    uint32_t sa, alo, ahi;
                    const float rcp[1] = {w4_group_rcp(ta, sa)};
                    const float(*const runs[1])[8] = {&ta};
                    w4_run48(w4_codes<1>(runs, rcp), 0, alo, ahi);
                    w4.put(stage, alo, ahi, sa);
                }
                if (lane < kStageLanes)
                    buffer_store_b128<0>(__builtin_bit_cast(buffer_u32x4, *reinterpret_cast<const uint4 *>(stage + vstage)), rs_c, vout, group(i) * (p.Mpad / 32) * kW4ABlock);
            }
        }
        if constexpr (RB > 0) {
            // only this wavefront touches its block, and the LDS queue of a wavefront is in order: no barrier
            *reinterpret_cast<uint4 *>(block + r8 * L::kXRow + 16 * c8) = xa[i % kX];
            if (kTwo) *reinterpret_cast<uint4 *>(block + (r8 + 8) * L::kXRow + 16 * c8) = xb[i % kX];
            const uint4 *ap = reinterpret_cast<const uint4 *>(block + row % TOK * L::kXRow + 32 * blk);      // (of eight tokens: each twice)
            const uint4 x0 = ap[0], x1 = ap[1];
            const Frags now = fr;
            if (i + 1 < NG) fr = load_l1(i + 1);
#pragma unroll
            for (int c = 0; c < RB; ++c) {      // (a group past K: X is zero)
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x0), __builtin_bit_cast(bf16x8, now.b[2 * c]), acc[c], 0, 0, 0);
                acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x1), __builtin_bit_cast(bf16x8, now.b[2 * c + 1]), acc[c], 0, 0, 0);
            }
        }
        if constexpr (kX < NG) {
            __builtin_amdgcn_sched_barrier(0);
            if (i + kX < NG) load_x(i + kX);
        }
    }
    float *mx = reinterpret_cast<float *>(lds);      // INT8: [16 tokens][wavefronts]
    if constexpr (FMT == 2) {
        amax_a = max_over_8_lanes(amax_a);
        if (kTwo) amax_b = max_over_8_lanes(amax_b);
        if (c8 == 0) {
            mx[r8 * kWaves + wave] = amax_a;
            if (kTwo) mx[(r8 + 8) * kWaves + wave] = amax_b;
        }
    }
    if constexpr (RB > 0) {
        float *red = reinterpret_cast<float *>(block);
#pragma unroll
        for (int c = 0; c < RB; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[(4 * blk + v) * L::kRedRow + 16 * c + row] = acc[c][v];
    }
    __syncthreads();

    if constexpr (FMT == 2) {
        // Eq. 1 with q_max = 127: s = fp16(max / 127) (IEEE division, round to nearest even, saturating), codes from x^ * (1.0f / s)
        auto token_max = [&](int t) {
            const float4 *q = reinterpret_cast<const float4 *>(mx + t * kWaves);
            float m = 0.f;
#pragma unroll
            for (int k = 0; k < kWaves / 4; ++k) m = fmaxf(fmaxf(m, fmaxf(q[k].x, q[k].y)), fmaxf(q[k].z, q[k].w));
            return m;
        };
        auto scale_of = [](float amax, _Float16 &sh) {
            float s32 = amax / 127.0f;
            s32 = fminf(s32, 65504.0f);
            sh = (_Float16)s32;
            const float sc = (float)sh;
            return sc > 0.f ? 1.0f / sc : 0.f;
        };
        _Float16 sha, shb = 0;
        const float rcp_a = scale_of(token_max(r8), sha), rcp_b = kTwo ? scale_of(token_max(r8 + 8), shb) : 0.f;
        if (wave == 0 && c8 == 0) {      // rows past M: padding entries of the scale vector (it has Mpad of them)
            p.sx[ma] = __builtin_bit_cast(uint16_t, sha);
            if (kTwo) p.sx[mb] = __builtin_bit_cast(uint16_t, shb);
        }
        if (!kKeep) {
            // (or the compiler keeps what the first walk loaded and unpacked for the second, and spills it)
            asm volatile("" : "+v"(vr));
#pragma unroll
            for (int i = 0; i < NG; ++i)      // (sixteen tokens: fewer are kept as x^)
                asm volatile("" : "+v"(xa[i].x), "+v"(xa[i].y), "+v"(xa[i].z), "+v"(xa[i].w), "+v"(xb[i].x), "+v"(xb[i].y), "+v"(xb[i].z), "+v"(xb[i].w));
        }
        auto codes = [&](const float (&x)[8], float rcp) {
            // 1.5 * 2^23 added: the sum is rounded to a whole number (to nearest, ties to even) and has it in its low bits
            uint32_t w[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) w[e] = __float_as_uint(__builtin_amdgcn_fmed3f(x[e] * rcp, -127.f, 127.f) + 0x1.8p23f);
            auto low4 = [](uint32_t a, uint32_t b, uint32_t c, uint32_t d) {
                return (uint32_t)__builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, 0x0c0c0400), __builtin_amdgcn_perm(b, a, 0x0c0c0400), 0x05040100);
            };
            return u32x2{low4(w[0], w[1], w[2], w[3]), low4(w[4], w[5], w[6], w[7])};
        };
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            if (!kKeep) {
                __builtin_amdgcn_sched_barrier(0);
                if (i == 0) { load_rinv(0); load_rinv(1); }
                else if (i + 1 < NG) load_rinv(i + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (group(i) < p.G) {
                float ta[8], tb[8];
                if (!kKeep) {
                    smooth(xa[i % kX], r0[i], r1[i], ta);
                    smooth(xb[i % kX], r0[i], r1[i], tb);
                }
                const int sc = group(i) * p.Mpad * 64;      // a group is two 32-channel steps of operand blocks
                __builtin_amdgcn_raw_buffer_store_b64(codes(kKeep ? keep[kKeep ? i : 0][0] : ta, rcp_a), rs_c, vca, sc, 0);
                if (kTwo) __builtin_amdgcn_raw_buffer_store_b64(codes(kKeep ? keep[kKeep ? i : 0][TOK / 8 - 1] : tb, rcp_b), rs_c, vcb, sc, 0);
            }
        }
    }

    // housekeeping for the kernel that follows on the stream: its tile arrival counters start at zero
    for (int i = blockIdx.x * (kWaves * 64) + threadIdx.x; i < p.n_zero; i += gridDim.x * (kWaves * 64)) p.zero_words[i] = 0u;

    if constexpr (RB > 0) {
        // the wavefronts' partial H, added in wavefront order; a thread takes two neighbouring columns of one token
        const int pairs = p.rank / 2;
        for (int idx = threadIdx.x; idx < TOK * pairs; idx += kWaves * 64) {
            const int r = idx / pairs, col = 2 * (idx - r * pairs);
            float h0 = 0.f, h1 = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const float *q = reinterpret_cast<const float *>(lds + L::kMax + w * L::kWave) + r * L::kRedRow + col;
                h0 += q[0];
                h1 += q[1];
            }
            const int m = m0 + r;       // < Mpad: rows past M land in padding
            *reinterpret_cast<float2 *>(p.H + (size_t)m * p.rank + col) = make_float2(h0, h1);
            const uint32_t hi = bf16_rne_pair(h0, h1), lo = bf16_rne_pair(h0 - bf16lo(hi), h1 - bf16hi(hi));
            *reinterpret_cast<uint32_t *>(p.hfrag + hfrag_offset(p.rank, m, col, 0) + (col % 8) * 2) = hi;
            *reinterpret_cast<uint32_t *>(p.hfrag + hfrag_offset(p.rank, m, col, 1) + (col % 8) * 2) = lo;
        }
    }
}

// Tokens of a workgroup: eight while those are one round of the CUs.  The operand rows past the eight repeat them, and the L1 fragments
// are read for half as many tokens, which is the smaller part.  us per forward, 16 tokens -> 8, same bits: INT8 M = 1337, K = 3072, N = 9216, rank 16 49.5 -> 46.7,
// M = 1024, K = 1152, N = 4608 18.4 -> 17.2, M = 2000, K = N = 3072 34.7 -> 32.4, M = 2048, K = 640, N = 9216, rank 32 30.7 -> 29.5; MXFP4 M = 1500, K = 6144, N = 3072,
// rank 32 38.9 -> 35.5, M = 2048, K = N = 3072 25.8 -> 24.8, M = 1024, K = 1152, N = 4608 15.6 -> 15.1; INT4 M = 2048, K = 4608, N = 1152 34.1 -> 32.2, M = 1337, K = 3072, N = 9216,
// rank 16 55.5 -> 54.3, M = 1800, K = 1536, N = 9216 52.9 -> 52.7.
int act_one_pass_tokens(int M) { return (M + 7) / 8 <= 256 ? 8 : 16; }

template <int FMT, int RB, int NG, int TOK>
hipError_t launch_tokens(const ActParams &p, hipStream_t stream) {
    auto k = act_onepass_kernel<FMT, RB, NG, TOK>;
    constexpr int bytes = OnePassLds<RB>::kBytes;
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), bytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)((p.M + TOK - 1) / TOK)), dim3(kWaves * 64), bytes, stream, p);
    return hipGetLastError();
}

template <int FMT, int RB, int NG>
hipError_t launch_one(const ActParams &p, hipStream_t stream) {
    if constexpr (FMT == 1 && RB == 4) return launch_tokens<FMT, RB, NG, 8>(p, stream);
    else return act_one_pass_tokens(p.M) == 8 ? launch_tokens<FMT, RB, NG, 8>(p, stream) : launch_tokens<FMT, RB, NG, 16>(p, stream);
}

template <int FMT, int RB>
hipError_t launch_groups(const ActParams &p, hipStream_t stream) {
    if (p.G <= 32) return launch_one<FMT, RB, 2>(p, stream);
    if (p.G <= 48) return launch_one<FMT, RB, 3>(p, stream);
    if constexpr (RB <= 2) return launch_one<FMT, RB, 6>(p, stream);
    return hipErrorInvalidValue;
}

template <int FMT>
hipError_t launch_rank(const ActParams &p, int flags, hipStream_t stream) {
    if (!(flags & 2) || p.rank == 0) return launch_groups<FMT, 0>(p, stream);
    if (p.rank <= 16) return launch_groups<FMT, 1>(p, stream);
    if (p.rank <= 32) return launch_groups<FMT, 2>(p, stream);
    if constexpr (FMT != 0) return launch_groups<FMT, 4>(p, stream);
    return hipErrorInvalidValue;
}

}  // namespace

// Which calls take this kernel.  us per forward, act_kernel.hip -> this one:
// INT8: everything whose K fits the registers (six groups per wavefront up to rank 32, three up to rank 64), except short rows in
// more than one round of workgroups (M = 4608, K = 1152, rank 64: 42.0 -> 42.8) and rows of at most eight groups, which leave half of
// the wavefronts without one (1 to 4000 tokens: 1 to 13 % slower than the walking kernel at up to eight groups, 1 to 6 % faster from
// nine on).  M = 1, K = 3072, N = 9216 15.7 -> 14.2; M = 300,
// K = 3072, N = 2064 22.4 -> 17.9; M = 2048, K = N = 3072 40.4 -> 34.6; M = 4608, K = N = 3072 69.7 -> 64.1.
// INT4 and MXFP4, whose groups do not wait for each other: what act_pass_instead names (layout.h), and else one round of workgroups that fills a quarter of the CUs at
// least; fewer slices do better with K cut into runs, a second round undoes the gain.  INT4: M = 1337, K = 3072, N = 9216
// 61.5 -> 60.0, M = 4096, K = 6144, N = 2048 80.5 -> 78.2, M = 4608, K = 3072, N = 3072 65.3 -> 67.8; MXFP4: M = 2048, K = N = 3072
// 28.7 -> 27.5, M = 4608, K = 6144, N = 3072 72.4 -> 75.3; INT4 at rank 64: no difference.
// MXFP4 with eight tokens to a workgroup, act_tile_kernel.hip -> this one: K = 1024 (below, partial H is left to the GEMM: layout.h, act_pass_instead) to 3072 from 241 tokens on, M = 270, K = 1152, N = 12288, rank 32
// 16.4 -> 13.8, M = 397, K = 2240, N = 10208 21.0 -> 19.2, and ranks 48 and 64 (layout.h, plan_act_tile); longer rows hold six groups per wavefront, and few or
// wide ones lose: M = 526, K = 3712, N = 7392, rank 32 24.0 | 25.3, M = 1500, K = 6144, N = 3072, rank 64 38.0 | 41.4.  INT4 (spilled registers at rank 64): M = 905, K = 3136,
// N = 5264, rank 48 38.0 | 43.7.  Without a branch cut runs cost no second launch (act_kernel.hip | this): M = 667, K = 3008, N = 64 9.5 | 10.2, M = 300, K = 2240, N = 2800 8.6 | 8.9, M = 500,
// K = 3072, N = 6400 16.1 | 17.1; M = 257, K = 1024, N = 3072 9.6 | 9.3, M = 1000, K = 1536, N = 1024 10.4 | 10.1.
bool act_one_pass(int fmt, int M, int K, int rank) {
    const int G = K / kGroup, slices = (M + 15) / 16;
    if (fmt == 1 && G >= 16 && G <= 3 * kWaves && act_one_pass_tokens(M) == 8) return slices >= (rank > 0 || G <= 24 ? 16 : 64) && rank <= 64;
    if (fmt == 0 && act_pass_instead(true, M, 0, G, rank, 0)) return true;
    if (fmt != 2) return slices >= 64 && slices <= 256 && G <= 6 * kWaves && rank <= 32;
    if (G <= 8 || (slices > 256 && G <= 24)) return false;
    return (G <= 3 * kWaves && rank <= 64) || (G <= 6 * kWaves && rank <= 32);
}

hipError_t launch_act_one_pass(const ActParams &p, int flags, hipStream_t stream) {
    if (p.M <= 0) return hipSuccess;
    if (!act_one_pass(p.fmt, p.M, p.K, p.rank) || !(flags & 1) || (p.fmt != 0 && !p.sx) || p.K != p.G * kGroup || p.rank % 16 ||
        (size_t)p.K * p.Mpad >= ((size_t)1 << 31))
        return hipErrorInvalidValue;
    return p.fmt == 2 ? launch_rank<2>(p, flags, stream) : p.fmt == 1 ? launch_rank<1>(p, flags, stream) : launch_rank<0>(p, flags, stream);
}

}  // namespace svdq
