// W4A4 GEMM for launches of few output tiles (small batches, narrow layers): the arithmetic of gemm_w4a4_kernel.hip
// (exact group sums from the block-scaled MFMA, scale tiles from an f16 MFMA, one FMA per partial sum; arXiv 2411.05007
// Eq. 5), another division of the work.
//
// Such a launch is bound by one tile's chain of K steps - the 128 x 256 tiles of gemm_w4a4_kernel.hip leave most CUs
// idle, walk K behind a barrier per group, and a K loop split over workgroups parks its partial tiles past the L2.  Here a workgroup owns a small
// tile, (32 RB) x 64, and its four or eight wavefronts share the tile's K, each taking every KS-th group: operands go
// from the L2 straight into the registers the MFMAs read (one weight block and RB activation blocks per group and
// wavefront, requested one or two groups ahead, each as soon as its registers are free), nobody waits for anybody in
// the loop, and the partial tiles meet once, in LDS.  Bound: a lone launch by its fixed parts (start, first
// operands, low-rank product, the meeting: 5 to 6 us together), larger ones by the operands' way from the L2 (by counters 375
// MB at M = 512, K = 3072, N = 9216, 13 TB/s; 511 MB at M = 4096, K = 4608, N = 1152, 15 TB/s).  us of the GEMM in a kernel trace,
// before -> after: M = 256, K = N = 1152 20.5 -> 5.8; M = 300, K = 3072, N = 2064 26.4 -> 8.6; M = 512, K = 3072, N = 9216 31.7 -> 28.3;
// M = 512, K = 12288, N = 3072 45.0 -> 27.1; M = 4096, K = 4608, N = 1152 41.1 -> 34.8.  The variants' limits: layout.h, plan_kpar_int4.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "buffer.h"
#include "gemm_common.h"
#include "gemm_kpar.h"
#include "kernels.h"
#include "layout.h"
#include "lds_limit.h"

namespace svdq {
namespace {

typedef int intx8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int kFmtE2M3 = 2;                 // operand format selector of the instruction
constexpr int kScaleBytes = 0x8082;         // block scales 2^3 and 2^1, as in gemm_w4a4_kernel.hip

// RB row blocks of 32, KS wavefronts that share K, DEPTH groups requested ahead; RUNS: H comes as the partial sums of the
// activation kernel's runs (else ready-made)
template <int RB, int KS, int DEPTH, bool RUNS>
__global__ __launch_bounds__(KS * 64, KS == 8 ? 1 : 2) void gemm_w4a4_kpar_kernel(GemmW4Params p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int CB = 2;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31;
    const int tiles_m = (p.M + 32 * RB - 1) / (32 * RB), tiles_n = (p.N + 63) / 64;
    int tile_m, tile_n;
    kpar_tile_of((int)blockIdx.x, tiles_m, tiles_n, RB * kW4ABlock, kW4BBlock, tile_m, tile_n);
    const int gm0 = tile_m * 32 * RB, gn0 = tile_n * 64;      // the launch checks that every tile lies inside the padded rows and columns

    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.xa, w4_a_bytes(p.G, p.Mpad));
    const __amdgpu_buffer_rsrc_t rs_b = make_rsrc(p.wb, w4_b_bytes(p.G, p.Npad));
    const int a_stride = (p.Mpad / 32) * kW4ABlock, b_stride = (p.Npad / 64) * kW4BBlock;      // bytes per group
    const int a_base = (gm0 / 32) * kW4ABlock, b_base = (gn0 / 64) * kW4BBlock;
    const int n = wave < p.G ? (p.G - wave + KS - 1) / KS : 0;      // this wavefront's groups: wave, wave + KS, ...
    auto group_of = [&](int i) { return wave + KS * (i < n ? i : n - 1); };      // past the end: the last one again, loaded and ignored
    const int va = 24 * lane, vb = 16 * lane, vsx = kW4ACodes + 4 * li, vsw = kW4BCodes + 4 * li;

    struct ASet { u32x4 lo[RB]; u32x2 hi[RB]; uint32_t sx[RB]; };
    struct BSet { u32x4 q[CB]; uint32_t sw[CB]; };
    struct BFrag { uint32_t d[6]; };
    ASet A[DEPTH];
    BSet B[DEPTH];
    auto load_a = [&](ASet &s, int r, int i) {
        const int off = a_base + r * kW4ABlock + group_of(i) * a_stride;
        s.lo[r] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_a, va, off, 0));
        s.hi[r] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rs_a, va + 16, off, 0));
    };
    auto load_sx = [&](ASet &s, int r, int i) { s.sx[r] = __builtin_amdgcn_raw_buffer_load_b32(rs_a, vsx, a_base + r * kW4ABlock + group_of(i) * a_stride, 0); };
    auto load_b = [&](BSet &s, int c, int i) {
        s.q[c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_b, vb, b_base + c * 1024 + group_of(i) * b_stride, 0));
    };
    auto load_sw = [&](BSet &s, int c, int i) { s.sw[c] = __builtin_amdgcn_raw_buffer_load_b32(rs_b, vsw, b_base + c * 128 + group_of(i) * b_stride, 0); };
    // the six operand registers of 32 weight codes from their four stored registers (layout.h)
    auto expand = [&](BFrag &f, u32x4 q) {
        f.d[0] = q.x & ~kW4Z0;
        f.d[1] = q.y & ~kW4Z1;
        f.d[2] = (q.x & kW4Z0) | (q.y & kW4Z1);
        f.d[3] = q.z & ~kW4Z0;
        f.d[4] = q.w & ~kW4Z1;
        f.d[5] = (q.z & kW4Z0) | (q.w & kW4Z1);
        // (made here and now: sunk to its first use, behind the refill of q, it would keep the old words alive beside the new)
        asm volatile("" : "+v"(f.d[0]), "+v"(f.d[1]), "+v"(f.d[2]), "+v"(f.d[3]), "+v"(f.d[4]), "+v"(f.d[5]));
    };
    // A scale dword (fp16 scale, zero high half) in both registers of the f16 MFMA's operand, as in gemm_w4a4_kernel.hip.
    // Two moves of their own: a pair that shared a register with the word it was made from would keep the next group's
    // word from being loaded into its place.
    auto pair_of = [&](uint32_t s) {
        u32x2 x;
        uint32_t lo, hi;
        asm volatile("v_mov_b32 %0, %1" : "=v"(lo) : "v"(s));
        asm volatile("v_mov_b32 %0, %1" : "=v"(hi) : "v"(s));
        x.x = lo;
        x.y = hi;
        return x;
    };
    auto op_a = [&](const ASet &s, int r) { return intx8{(int)s.lo[r].x, (int)s.lo[r].y, (int)s.lo[r].z, (int)s.lo[r].w, (int)s.hi[r].x, (int)s.hi[r].y, 0, 0}; };
    auto op_b = [&](const BFrag &f) { return intx8{(int)f.d[0], (int)f.d[1], (int)f.d[2], (int)f.d[3], (int)f.d[4], (int)f.d[5], 0, 0}; };
    auto op_s = [&](u32x2 x) { return __builtin_bit_cast(halfx4, x); };
    const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int scales = kScaleBytes;
    asm volatile("" : "+v"(scales));      // one vector register for good (the scale operand cannot be a constant)

    if (n > 0) {
#pragma unroll
        for (int s = 0; s < DEPTH; ++s) {
#pragma unroll
            for (int c = 0; c < CB; ++c) { load_b(B[s], c, s); load_sw(B[s], c, s); }
#pragma unroll
            for (int r = 0; r < RB; ++r) { load_a(A[s], r, s); load_sx(A[s], r, s); }
        }
    }
    __builtin_amdgcn_sched_barrier(0);      // the first operands are requested before H and L2

    // bias (wavefront 0) and low-rank product (rank step ks by wavefront ks % KS)
    float acc[RB][CB][16];
    {
        floatx16 lr[RB][CB];
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            const float b = wave == 0 ? p.bias[gn0 + c * 32 + li] : 0.f;      // padded to Npad
#pragma unroll
            for (int r = 0; r < RB; ++r) lr[r][c] = floatx16{b, b, b, b, b, b, b, b, b, b, b, b, b, b, b, b};
        }
        if constexpr (RUNS) {
            // L2's operands of the wavefront's first rank step are requested before H is added up
            GemmLowRankStep<RB, CB> o;
            if (wave < p.rank / 16) gemm_lowrank_load_l2<RB, CB>(o, p.l2t, p.rank, gn0, lane, wave);
            kpar_sum_h_tile<RB, KS>(lds, p.hpart, p.runs, p.M, p.Mpad, p.rank, gm0, threadIdx.x);
            for (int ks = wave; ks < p.rank / 16; ks += KS) {
                if (ks != wave) gemm_lowrank_load_l2<RB, CB>(o, p.l2t, p.rank, gn0, lane, ks);
                gemm_lowrank_load_h<RB, CB>(o, lds + lane * 16, p.rank, ks);
                gemm_lowrank_multiply<RB, CB>(lr, o);
            }
        } else {
            for (int ks = wave; ks < p.rank / 16; ks += KS) {
                GemmLowRankStep<RB, CB> o;
                gemm_lowrank_load<RB, CB>(o, p.hfrag + (size_t)(gm0 / 32) * (p.rank / 16) * 2048 + lane * 16, p.l2t, p.rank, gn0, lane, ks);
                gemm_lowrank_multiply<RB, CB>(lr, o);
            }
        }
#pragma unroll
        for (int r = 0; r < RB; ++r)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[r][c][v] = lr[r][c][v];
    }

    BFrag bf[CB];
    u32x2 sxp, swp[CB];
    floatx16 ag[2], sg;
// (empty asm statements that "rewrite" a register pin the order, as in gemm_w4a4_kernel.hip)
#define KP_SB() __builtin_amdgcn_sched_barrier(0)
#define KP_MFMA_A(DST, ASET, R, BF)                                                                                                     \
    DST = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(op_a(ASET, R), op_b(BF), zero16, kFmtE2M3, kFmtE2M3, 0, scales, 1, scales);   \
    asm volatile("" : "+v"(DST), "+v"(sg))
#define KP_MFMA_S(R, C, SX, SW)                                                         \
    asm volatile("" : "+v"(acc[R][C][0]), "+v"(acc[R][C][15]), "+v"(SX));               \
    sg = __builtin_amdgcn_mfma_f32_32x32x8f16(op_s(SX), op_s(SW), zero16, 0, 0, 0);     \
    asm volatile("" : "+v"(sg))
    if (n > 0) {
#pragma unroll
        for (int c = 0; c < CB; ++c) { expand(bf[c], B[0].q[c]); swp[c] = pair_of(B[0].sw[c]); }
        sxp = pair_of(A[0].sx[0]);
        KP_SB();
#pragma unroll
        for (int c = 0; c < CB; ++c) { load_b(B[0], c, DEPTH); load_sw(B[0], c, DEPTH); }
        load_sx(A[0], 0, DEPTH);
        KP_SB();
        sg = zero16;
        KP_MFMA_A(ag[0], A[0], 0, bf[0]);
        sg = __builtin_amdgcn_mfma_f32_32x32x8f16(op_s(sxp), op_s(swp[0]), zero16, 0, 0, 0);
        asm volatile("" : "+v"(sg));
        KP_SB();
        // group i in 2 RB slots t = 2 r + c: group-sum MFMA of the next block | the sixteen FMAs of this block | scale-tile
        // MFMA of the next block; whatever has been used for the last time is requested again at once, DEPTH groups on
        auto body = [&](int i, auto set_tag) {
            constexpr int S = decltype(set_tag)::value, S1 = (S + 1) % DEPTH;
#pragma unroll
            for (int t = 0; t < 2 * RB; ++t) {
                const int r = t / 2, c = t % 2;
                constexpr int last = 2 * RB - 1;
                const int r1 = t == last ? 0 : (t + 1) / 2, c1 = (t + 1) % 2;
                KP_SB();
                if (t == last) { KP_MFMA_A(ag[(t + 1) & 1], A[S1], r1, bf[c1]); }
                else { KP_MFMA_A(ag[(t + 1) & 1], A[S], r1, bf[c1]); }
                if (c1 == 1) load_a(A[S], r1, i + DEPTH);            // row block r1 of this group has been multiplied for the last time
                if (t >= 2 * RB - 2) {                               // so has column block c: the next group's takes its place
                    expand(bf[c], B[S1].q[c]);
                    load_b(B[S1], c, i + 1 + DEPTH);
                }
                KP_SB();
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[r][c][v] = __builtin_fmaf(ag[t & 1][v], sg[v], acc[r][c][v]);
                KP_SB();
                if (t == last) {
#pragma unroll
                    for (int cc = 0; cc < CB; ++cc) { swp[cc] = pair_of(B[S1].sw[cc]); load_sw(B[S1], cc, i + 1 + DEPTH); }
                    sxp = pair_of(A[S1].sx[0]);
                    load_sx(A[S1], 0, i + 1 + DEPTH);
                } else if (c1 == 0) {
                    sxp = pair_of(A[S].sx[r1]);
                    load_sx(A[S], r1, i + DEPTH);
                }
                KP_MFMA_S(r, c, sxp, swp[c1]);
                KP_SB();
            }
        };
        static_assert(DEPTH == 1 || DEPTH == 2, "");
        for (int i = 0; i < n; i += DEPTH) {
            body(i, std::integral_constant<int, 0>{});
            if constexpr (DEPTH > 1) {
                if (i + 1 >= n) break;
                body(i + 1, std::integral_constant<int, 1 % DEPTH>{});
            }
        }
    }
    if constexpr (RUNS) __syncthreads();      // nobody reads H any more
    kpar_reduce_store<RB, CB, KS>(acc, lds, p.Y, p.M, p.N, gm0, gn0, wave, lane);
}

template <int RB, int KS, int DEPTH, bool RUNS>
hipError_t launch_variant(const GemmW4Params &p, hipStream_t stream) {
    const int tiles_m = (p.M + 32 * RB - 1) / (32 * RB), tiles_n = (p.N + 63) / 64;
    // H, L2 and the bias are read with plain loads: every tile must lie inside the padded rows and columns
    if (tiles_m * 32 * RB > p.Mpad || tiles_n * 64 > p.Npad) return hipErrorInvalidValue;
    auto k = gemm_w4a4_kpar_kernel<RB, KS, DEPTH, RUNS>;
    constexpr int bytes = KparLds<RB, 2, KS>::kBytes;
    if (RUNS && (!p.hpart || p.rank <= 0 || kpar_h_bytes<RB>(p.rank) > bytes)) return hipErrorInvalidValue;
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), bytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(tiles_m * tiles_n), dim3(KS * 64), bytes, stream, p);
    return hipGetLastError();
}

template <int RB, int KS, int DEPTH>
hipError_t launch_kpar(const GemmW4Params &p, hipStream_t stream) {
    return p.runs > 0 ? launch_variant<RB, KS, DEPTH, true>(p, stream) : launch_variant<RB, KS, DEPTH, false>(p, stream);
}

}  // namespace

hipError_t launch_gemm_w4a4_kpar(const GemmW4Params &p, hipStream_t stream) {
    if (p.ksplit != 1 || p.dbg) return hipErrorInvalidValue;
    switch (p.kpar) {
        case kKpar1x8: return launch_kpar<1, 8, 2>(p, stream);
        case kKpar2x8: return launch_kpar<2, 8, 1>(p, stream);
        case kKpar2x4: return launch_kpar<2, 4, 2>(p, stream);
        case kKpar4x8: return launch_kpar<4, 8, 1>(p, stream);
        case kKpar4x4: return launch_kpar<4, 4, 1>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace svdq
