// MXFP4 and INT8 GEMMs for launches of few output tiles (small batches, narrow layers): the arithmetic of
// gemm_fp4_kernel.hip and w8a8_kernels.hip (arXiv 2411.05007 Eq. 5), the division of the work of
// gemm_w4a4_kpar_kernel.hip.  A workgroup owns a small tile, (32 RB) x 64 or 32 x 32 (CB = 1); its four, eight or (32 x 32 tiles) sixteen
// wavefronts share the tile's K, wavefront w taking steps w, w + KS, ...  Both formats store a 32-row block of one step (64 channels
// of MXFP4, 32 of INT8) as one contiguous kilobyte in operand order, so a step is RB + CB loads of 16 bytes per lane straight into the
// registers that the RB CB MFMAs read, DEPTH steps ahead; nobody waits for anybody in the loop, and the partial tiles meet
// once, in LDS.  Bound: one image row by the weights' way from memory (M = 16, K = N = 12288: 75 MB of MXFP4 codes in a forward
// of 24 us), larger launches by the operands' way from the L2.  us of the GEMM in a kernel trace, before -> after, MXFP4:
// M = 512, K = N = 3072 18.7 -> 12.6; the rule that picks a variant, with more shapes: layout.h, plan_kpar_blocks.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "buffer.h"
#include "gemm_common.h"
#include "gemm_kpar.h"
#include "kernels.h"
#include "layout.h"
#include "lds_limit.h"

namespace svdq {
namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));
typedef int intx8 __attribute__((ext_vector_type(8)));
typedef int intx16 __attribute__((ext_vector_type(16)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int kFmtE2M1 = 4;                  // operand format selector of the instruction
constexpr int kRowBytes = 32;                // bytes of one row of one step, both formats

// what the two formats' launches have in common
struct KparParams {
    const uint8_t *xcodes, *wcodes;      // [step][rows / 32][64 lanes][16 bytes]
    const uint8_t *bx, *bw;              // MXFP4: scale bytes (layout.h)
    const uint16_t *sx, *sw;             // INT8: fp16 scales per token and per output channel
    const uint8_t *hfrag;
    const uint16_t *l2t;
    const float *bias;
    uint16_t *Y;
    int M, N, steps, Mpad, Npad, rank;
    const float *hpart;      // runs > 0: partial H of the activation kernel's runs, else hfrag holds the whole H
    int runs;
};

// I8: INT8 (32 channels per step), else MXFP4 (64).  RB row blocks and CB column blocks of 32, KS wavefronts that share K, DEPTH steps ahead.
// RUNS: H comes as the partial sums of the activation kernel's runs (else ready-made).  WALK (INT8): a way out behind every step of the K loop.
template <bool I8, int RB, int CB, int KS, int DEPTH, bool WALK, bool RUNS>
__global__ __launch_bounds__(KS * 64, KS >= 8 ? 1 : 2) void gemm_kpar_blocks_kernel(KparParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    using T = KparLds<RB, CB, KS>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lh = lane >> 5;
    const int tiles_m = (p.M + 32 * RB - 1) / (32 * RB), tiles_n = (p.N + 32 * CB - 1) / (32 * CB);
    int tile_m, tile_n;
    kpar_tile_of((int)blockIdx.x, tiles_m, tiles_n, RB * 1024, CB * 1024, tile_m, tile_n);
    const int gm0 = tile_m * 32 * RB, gn0 = tile_n * 32 * CB;      // the launch checks that every tile lies inside the padded rows and columns

    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.xcodes, (size_t)p.steps * p.Mpad * kRowBytes);
    const __amdgpu_buffer_rsrc_t rs_b = make_rsrc(p.wcodes, (size_t)p.steps * p.Npad * kRowBytes);
    const __amdgpu_buffer_rsrc_t rs_sa = make_rsrc(p.bx, I8 ? 0 : fp4_scale_bytes(p.steps, p.Mpad));
    const __amdgpu_buffer_rsrc_t rs_sb = make_rsrc(p.bw, I8 ? 0 : fp4_scale_bytes(p.steps, p.Npad));
    const int n = wave < p.steps ? (p.steps - wave + KS - 1) / KS : 0;      // this wavefront's steps

    static_assert(KS % 4 == 0, "");
    struct Set { u32x4 a[RB], b[CB]; uint32_t sa[I8 ? 1 : RB], sb[I8 ? 1 : CB]; };
    Set S[DEPTH];
    auto load = [&](Set &s, int i) {
        // past the end of the wavefront's steps: a lane offset beyond every buffer, which loads zeros and asks the memory for nothing
        const int past = i < n ? 0 : (int)0x80000000u;      // (every buffer is smaller than 2^31 bytes)
        const int st = kpar_step(wave, KS, i, n);
        const int va = lane * 16 + past, vs = lane * 4 + past;
        const int oa = (st * p.Mpad + gm0) * kRowBytes, ob = (st * p.Npad + gn0) * kRowBytes;
#pragma unroll
        for (int c = 0; c < CB; ++c) s.b[c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_b, va, ob + c * 1024, 0));
#pragma unroll
        for (int r = 0; r < RB; ++r) s.a[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_a, va, oa + r * 1024, 0));
        if constexpr (!I8) {
            // (whole dwords, which hold the bytes of four steps: of a byte's load the compiler masks the result, at the top of the K loop
            // for all sets at once)
            const int osa = (st >> 2) * p.Mpad * 8 + gm0 * 8, osb = (st >> 2) * p.Npad * 8 + gn0 * 8;
#pragma unroll
            for (int c = 0; c < CB; ++c) s.sb[c] = __builtin_amdgcn_raw_buffer_load_b32(rs_sb, vs, osb + c * 256, 0);
#pragma unroll
            for (int r = 0; r < RB; ++r) s.sa[r] = __builtin_amdgcn_raw_buffer_load_b32(rs_sa, vs, osa + r * 256, 0);
        }
    };
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) {
        load(S[d], d);
        // the first operands are requested before H and L2, and one step's before the next one's: mixed here, the wait at the top of the
        // K loop, which is the same for its first and every later round, is one for all of them
        __builtin_amdgcn_sched_barrier(0);
    }

    if constexpr (I8) {
        // What Eq. 2 and the 16-bit branch need of this wavefront's share of the outputs, requested while the first
        // operands are on their way: the scales, the bias, and the operands of rank step 0.  The share's kOPW octets of rows
        // lie in one row block; operand lane l feeds row l % 8 of octet l / 8 % kOPW, so that the first kOPW register quads of
        // the 32 x 32 product are the share's rows.
        typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
        constexpr int kPhases = RB / T::kPR;
        const int ksteps = p.rank / 16;
        int oct0, c0;
        kpar_share<RB, CB, KS>(wave % T::kActive, 0, oct0, c0);
        uint2 sx[kPhases][T::kOPW];
        float sw[T::kCPW], bias[T::kCPW];
        struct RankH { uint4 hi, lo; };
        struct RankL2 { uint4 b[T::kCPW]; };
        auto share_row = [&](int ph) { return (ph * T::kPR + oct0 / 4) * 32 + 8 * (oct0 % 4 + li / 8 % T::kOPW) + li % 8; };      // of the tile
        auto load_h = [&](RankH &o, int ph, int ks) {
            const unsigned char *h = p.hfrag + hfrag_offset(p.rank, gm0 + share_row(ph), 16 * ks + 8 * lh, 0);      // row < Mpad
            o.hi = *reinterpret_cast<const uint4 *>(h);
            o.lo = *reinterpret_cast<const uint4 *>(h + 1024);
        };
        auto load_l2 = [&](RankL2 &o, int ks) {
#pragma unroll
            for (int c = 0; c < T::kCPW; ++c) o.b[c] = *reinterpret_cast<const uint4 *>(p.l2t + (size_t)(gn0 + (c0 + c) * 32 + li) * p.rank + 16 * ks + 8 * lh);
        };
        // (H from runs: all of it is taken into registers here, its place in LDS is the partial tiles' later; at most two rank steps)
        constexpr int kEarly = RUNS ? 2 : 1;
        RankH first_h[kPhases][kEarly];
        RankL2 first_l2;
#pragma unroll
        for (int c = 0; c < T::kCPW; ++c) {
            sw[c] = (float)__builtin_bit_cast(_Float16, p.sw[gn0 + (c0 + c) * 32 + li]);      // padded to Npad
            bias[c] = p.bias[gn0 + (c0 + c) * 32 + li];
        }
#pragma unroll
        for (int ph = 0; ph < kPhases; ++ph)
#pragma unroll
            for (int k = 0; k < T::kOPW; ++k)
                sx[ph][k] = *reinterpret_cast<const uint2 *>(p.sx + gm0 + (ph * T::kPR + oct0 / 4) * 32 + 8 * (oct0 % 4 + k) + 4 * lh);      // < Mpad
        if (ksteps > 0) load_l2(first_l2, 0);
        if constexpr (RUNS) kpar_sum_h_tile<RB, KS>(lds, p.hpart, p.runs, p.M, p.Mpad, p.rank, gm0, threadIdx.x);
#pragma unroll
        for (int ph = 0; ph < kPhases; ++ph)
#pragma unroll
            for (int ks = 0; ks < kEarly; ++ks)
                if (ks < ksteps) {
                    if constexpr (RUNS) {
                        const unsigned char *h = lds + hfrag_offset(p.rank, share_row(ph), 16 * ks + 8 * lh, 0);
                        first_h[ph][ks].hi = *reinterpret_cast<const uint4 *>(h);
                        first_h[ph][ks].lo = *reinterpret_cast<const uint4 *>(h + 1024);
                    }
                    else load_h(first_h[ph][ks], ph, ks);
                }
        intx16 acc[RB][CB];
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[r][c] = intx16{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        auto multiply = [&](int d) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int c = 0; c < CB; ++c)
                    acc[r][c] = __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(intx4, S[d].a[r]), __builtin_bit_cast(intx4, S[d].b[c]), acc[r][c], 0, 0, 0);
        };
        // whole rounds of DEPTH steps without a way out between them (the compiler counts the requests on the shortest way to a set's use:
        // with one, every round began with a wait for all of them), then what is left, already requested.  us per forward before and
        // after: MXFP4, rank 32, M = 512, K = N = 3072 16.9 | 15.3, M = 1024 21.9 | 19.6, rank 64, M = 300, K = 6144, N = 4096 25.4 | 22.3
        if constexpr (WALK) {
            for (int i = 0; i < n; i += DEPTH) {
#pragma unroll
                for (int d = 0; d < DEPTH; ++d) {
                    if (d > 0 && i + d >= n) break;
                    multiply(d);
                    load(S[d], i + d + DEPTH);
                }
            }
        } else {
            int i = 0;
            for (; i + DEPTH <= n; i += DEPTH)
#pragma unroll
                for (int d = 0; d < DEPTH; ++d) {
                    multiply(d);
                    load(S[d], i + d + DEPTH);
                }
#pragma unroll
            for (int d = 0; d + 1 < DEPTH; ++d)
                if (i + d < n) multiply(d);
        }
        int f[RB][CB][16];
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) f[r][c][v] = acc[r][c][v];
        if constexpr (RUNS) __syncthreads();      // nobody reads H any more
        KparStore<RB, CB, KS> out(lds, wave, lane);
        floatx16 y[T::kCPW];
#pragma unroll
        for (int c = 0; c < T::kCPW; ++c) y[c] = floatx16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        // the scaled sums, the 16-bit branch and the bias in the order of the large-tile kernel: the same bits
        kpar_meet<RB, CB, KS>(f, lds, wave, lane,
            [&](int p0, int k, int c, Kpar4<int> s) {
                const uint2 raw = sx[p0 / T::kPR][k];
                const uint32_t w2[2] = {raw.x, raw.y};
                const int sum[4] = {s.x, s.y, s.z, s.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float sxe = (float)__builtin_bit_cast(_Float16, (uint16_t)(w2[e >> 1] >> (16 * (e & 1))));
                    y[c][4 * k + e] = (float)sum[e] * (sxe * sw[c]);
                }
            },
            [&](int p0) {
                RankH h = first_h[p0 / T::kPR][0];
                RankL2 l2 = first_l2;
                for (int ks = 0; ks < ksteps; ++ks) {
                    RankH next_h = first_h[p0 / T::kPR][kEarly - 1];
                    RankL2 next_l2 = l2;
                    if (ks + 1 < ksteps) {
                        load_l2(next_l2, ks + 1);
                        if (!RUNS) load_h(next_h, p0 / T::kPR, ks + 1);
                    }
#pragma unroll
                    for (int c = 0; c < T::kCPW; ++c) {
                        const bf16x8_t b = __builtin_bit_cast(bf16x8_t, l2.b[c]);
                        y[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, h.hi), b, y[c], 0, 0, 0);
                        y[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, h.lo), b, y[c], 0, 0, 0);
                    }
                    h = next_h;
                    l2 = next_l2;
                }
#pragma unroll
                for (int k = 0; k < T::kOPW; ++k)
#pragma unroll
                    for (int c = 0; c < T::kCPW; ++c)
                        out.put(k, c, Kpar4<float>{y[c][4 * k] + bias[c], y[c][4 * k + 1] + bias[c], y[c][4 * k + 2] + bias[c], y[c][4 * k + 3] + bias[c]});
                out.store(p0, p.Y, p.M, p.N, gm0, gn0);
            });
    } else {
        // bias (wavefront 0) and low-rank product (rank step ks by wavefront ks % KS) start the accumulators
        floatx16 acc[RB][CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const float b = wave == 0 ? p.bias[gn0 + c * 32 + li] : 0.f;      // padded to Npad
#pragma unroll
            for (int r = 0; r < RB; ++r) acc[r][c] = floatx16{b, b, b, b, b, b, b, b, b, b, b, b, b, b, b, b};
        }
        if constexpr (RUNS) {
            // L2's operands of the wavefront's first rank step are requested before H is added up
            GemmLowRankStep<RB, CB> o;
            if (wave < p.rank / 16) gemm_lowrank_load_l2<RB, CB>(o, p.l2t, p.rank, gn0, lane, wave);
            kpar_sum_h_tile<RB, KS>(lds, p.hpart, p.runs, p.M, p.Mpad, p.rank, gm0, threadIdx.x);
            for (int ks = wave; ks < p.rank / 16; ks += KS) {
                if (ks != wave) gemm_lowrank_load_l2<RB, CB>(o, p.l2t, p.rank, gn0, lane, ks);
                gemm_lowrank_load_h<RB, CB>(o, lds + lane * 16, p.rank, ks);
                gemm_lowrank_multiply<RB, CB>(acc, o);
            }
        } else {
            for (int ks = wave; ks < p.rank / 16; ks += KS) {
                GemmLowRankStep<RB, CB> o;
                gemm_lowrank_load<RB, CB>(o, p.hfrag + (size_t)(gm0 / 32) * (p.rank / 16) * 2048 + lane * 16, p.l2t, p.rank, gn0, lane, ks);
                gemm_lowrank_multiply<RB, CB>(acc, o);
            }
        }
        auto multiply = [&](int d) {
            __builtin_amdgcn_sched_barrier(0);
            int shift = (wave & 3) * 8;      // the wavefront's place in every chunk of four steps
            asm volatile("" : "+s"(shift));  // shifted here, not where the loads return
            auto op = [](u32x4 v) { return intx8{(int)v.x, (int)v.y, (int)v.z, (int)v.w, 0, 0, 0, 0}; };      // 4-bit formats: the first four registers
#pragma unroll
            for (int r = 0; r < RB; ++r)
#pragma unroll
                for (int c = 0; c < CB; ++c)
                    acc[r][c] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(op(S[d].a[r]), op(S[d].b[c]), acc[r][c], kFmtE2M1, kFmtE2M1,
                                                                               0, (int)(S[d].sa[I8 ? 0 : r] >> shift), 0, (int)(S[d].sb[I8 ? 0 : c] >> shift));
        };
        // (rounds as above; of two steps the second may be past the end and multiply zeros: a remainder's own copy of the registers spills)
        int i = 0;
        for (; DEPTH == 2 ? i < n : i + DEPTH <= n; i += DEPTH)
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                multiply(d);
                load(S[d], i + d + DEPTH);
            }
#pragma unroll
        for (int d = 0; d + 1 < DEPTH; ++d)
            if (DEPTH > 2 && i + d < n) multiply(d);
        float f[RB][CB][16];
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) f[r][c][v] = acc[r][c][v];
        if constexpr (RUNS) __syncthreads();      // nobody reads H any more
        kpar_reduce_store<RB, CB, KS>(f, lds, p.Y, p.M, p.N, gm0, gn0, wave, lane);
    }
}

template <bool I8, int RB, int CB, int KS, int DEPTH, bool WALK, bool RUNS>
hipError_t launch_tile(const KparParams &p, hipStream_t stream) {
    const int tiles_m = (p.M + 32 * RB - 1) / (32 * RB), tiles_n = (p.N + 32 * CB - 1) / (32 * CB);
    // H, L2, the scales and the bias are read with plain loads: every tile must lie inside the padded rows and columns
    if (tiles_m * 32 * RB > p.Mpad || tiles_n * 32 * CB > p.Npad) return hipErrorInvalidValue;
    auto k = gemm_kpar_blocks_kernel<I8, RB, CB, KS, DEPTH, WALK, RUNS>;
    constexpr int bytes = KparLds<RB, CB, KS>::kBytes;
    if (RUNS && (!p.hpart || p.rank <= 0 || (I8 && p.rank > 32) || kpar_h_bytes<RB>(p.rank) > bytes)) return hipErrorInvalidValue;
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), bytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(tiles_m * tiles_n), dim3(KS * 64), bytes, stream, p);
    return hipGetLastError();
}

template <bool I8, int RB, int CB, int KS, int DEPTH>
hipError_t launch_one(const KparParams &p, hipStream_t stream) {
    // INT8 on four wavefronts with a long K: us of the GEMM, rounds without a way out | a way out behind every step, rank 48: M = 700, N = 1824 (64-row
    // tiles): K = 640 5.8 | 6.2, 2048 9.7 | 9.6, 4608 16.4 | 15.4, 6080 21.0 | 19.0; M = 1464, N = 1520 (128-row): K = 2048 14.0 | 14.6, 3072 17.4 | 17.6,
    // 4608 23.2 | 21.7, 9600 43.9 | 39.8; 64-row tiles that add runs' H gain nothing (rank 16: K = 4608 16.2 | 17.0, 6080 20.2 | 19.7).  With eight wavefronts no
    // K was found where the rounds lose.
    if constexpr (I8 && KS == 4)
        if (p.steps > 128) {
            if (p.runs == 0) return launch_tile<I8, RB, CB, KS, DEPTH, true, false>(p, stream);
            if constexpr (RB == 4) return launch_tile<I8, RB, CB, KS, DEPTH, true, true>(p, stream);
        }
    return p.runs > 0 ? launch_tile<I8, RB, CB, KS, DEPTH, false, true>(p, stream) : launch_tile<I8, RB, CB, KS, DEPTH, false, false>(p, stream);
}

template <bool I8>
hipError_t launch_variant(const KparParams &p, int variant, hipStream_t stream) {
    switch (variant) {
        case kKparNarrow: return launch_one<I8, 1, 1, 16, 6>(p, stream);
        case kKpar1x8: return launch_one<I8, 1, 2, 8, 6>(p, stream);
        case kKpar2x8:      // (MXFP4 takes four wavefronts for 64-row tiles: plan_kpar_blocks)
            if constexpr (I8) return launch_one<true, 2, 2, 8, 4>(p, stream);
            return hipErrorInvalidValue;
        case kKpar2x4: return launch_one<I8, 2, 2, 4, 4>(p, stream);
        case kKpar4x8: return launch_one<I8, 4, 2, 8, 2>(p, stream);
        case kKpar4x4: return launch_one<I8, 4, 2, 4, 2>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_gemm_fp4_kpar(const GemmFp4Params &q, hipStream_t stream) {
    if (q.ksplit != 1) return hipErrorInvalidValue;
    KparParams p{};
    p.xcodes = q.xcodes; p.wcodes = q.wcodes; p.bx = q.bx; p.bw = q.bw;
    p.hfrag = q.hfrag; p.l2t = q.l2t; p.bias = q.bias; p.Y = q.Y;
    p.M = q.M; p.N = q.N; p.steps = q.G; p.Mpad = q.Mpad; p.Npad = q.Npad; p.rank = q.rank;
    p.hpart = q.hpart; p.runs = q.runs;
    return launch_variant<false>(p, q.kpar, stream);
}

hipError_t launch_gemm_w8a8_kpar(const GemmW8Params &q, hipStream_t stream) {
    if (q.ksplit != 1) return hipErrorInvalidValue;
    KparParams p{};
    p.xcodes = q.xcodes; p.wcodes = q.wcodes; p.sx = q.sx; p.sw = q.sw;
    p.hfrag = q.hfrag; p.l2t = q.l2t; p.bias = q.bias; p.Y = q.Y;
    p.M = q.M; p.N = q.N; p.steps = q.K / 32; p.Mpad = q.Mpad; p.Npad = q.Npad; p.rank = q.rank;
    p.hpart = q.hpart; p.runs = q.runs;
    return launch_variant<true>(p, q.kpar, stream);
}

}  // namespace svdq
