// Activation kernel, 32 tokens to a workgroup: the arithmetic of act_kernel.hip (arXiv 2411.05007 Sec. 4.3, Fig. 6b: "Quantize" and
// "Down Projection" share their input; Eq. 1 per group), for INT4 and MXFP4 launches whose K is cut into runs.
//
// The 16-token workgroups of act_kernel.hip read 16 KB of L1 fragments per 2 KB of X at rank 128, and where a launch's GEMM does not
// add up the runs' partial H they meet past the L2.  Here a wavefront takes a group of 32 tokens in the operand map of the 32 x 32 matrix
// instructions (lane l: token l % 32, channels 32 (l / 32) .. + 31), as fused_small_kernel.hip does: half the fragments per token, one
// reciprocal per lane instead of two, codes that come out as the GEMM's operand registers.  The four wavefronts of a workgroup share
// a run's groups, wavefront w taking groups w, w + 4, ..., with nothing to wait for in the loop; X is requested a group ahead, the
// fragments as soon as the products have read the last ones.  Their partial H meet in LDS and leave with plain stores, and
// act_sum_h_kernel adds the runs in order.
// us in a kernel trace, M = 512, K = 12288, rank 128: act_kernel.hip 16.9; this kernel 10.6 and the sum 4.8, of which the forward sees 12.6 (its start and end
// are shared with the neighbours').  Bound: a wavefront's chain (by counters 163 vector and 16 matrix instructions, 21 requests and two stores per
// group at rank 128, one wavefront per SIMD) and the fixed parts, 3 us of the 10.6.  Tried: the codes of a run kept in LDS and stored behind the loop (the same, but one workgroup per CU for long runs: M =
// 1800, K = 8192, N = 3072, rank 128 94.7 -> 97.7 us per forward); eight wavefronts (M = 512: 40.1 -> 40.6); parts that the GEMM adds (up to rank 64
// 2 to 10 % slower than act_kernel.hip's).  The rule, with both sides: layout.h, plan_act_tile.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "act_common.h"
#include "buffer.h"
#include "kernels.h"
#include "layout.h"
#include "lds_limit.h"

namespace svdq {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int WAVES = 4;
constexpr int kXRow = 144;                    // 128 bytes of a token's group + 16: the 32 rows of an operand read fall on distinct banks
constexpr int kOff = (int)0x80000000u;        // a lane offset beyond every buffer (layout.h, kpar_step): the load returns zeros

// LDS: the wavefronts' partial H, in whose places X is turned around (and the codes afterwards) and 1 / lambda of a group lies before
template <int RC> struct TileLds {
    static constexpr int kHRow = 32 * RC + 8;      // words; the two lane halves' rows, four apart, fall on different banks
    static constexpr int kTurn = 32 * kXRow + 256, kWave = 32 * kHRow * 4 > kTurn ? 32 * kHRow * 4 : kTurn, kBytes = WAVES * kWave;
    static_assert(2 * kBytes <= kLdsBytesPerCU, "");
};

// FMT 0: INT4, 1: MXFP4.  RC: blocks of 32 columns of H, zeros past the rank.  p.hpart: fp32 [run][M][rank]
template <int FMT, int RC>
__global__ __launch_bounds__(WAVES * 64, 2) void act_tile_kernel(ActParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    using L = TileLds<RC>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lh = lane >> 5;      // operand map: token li, channels 32 lh .. + 31 of the group
    const int tile = (int)blockIdx.x / p.chunks, run = (int)blockIdx.x - tile * p.chunks;
    const int gm0 = tile * 32, rows = p.M - gm0 < 32 ? p.M - gm0 : 32, rb = p.rank / 16;
    const int gbeg = run * p.gchunk, gend = gbeg + p.gchunk < p.G ? gbeg + p.gchunk : p.G;

    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.X, (size_t)p.M * p.K * 2);
    const __amdgpu_buffer_rsrc_t rs_r = make_rsrc(p.rinv, (size_t)p.K * 4);
    const __amdgpu_buffer_rsrc_t rs_l = make_rsrc(p.l1s, (size_t)p.K * p.rank * 2);
    const __amdgpu_buffer_rsrc_t rs_c = make_rsrc(p.codes, FMT == 1 ? (size_t)p.G * p.Mpad * kFp4RowBytes : w4_a_bytes(p.G, p.Mpad));
    const __amdgpu_buffer_rsrc_t rs_s = make_rsrc(p.sx, FMT == 1 ? fp4_scale_bytes(p.G, p.Mpad) : 0);
    // load map of X: request j reads tokens 8 j + lane / 8, channels 8 (lane % 8) .. + 7 of the group; rows past M read the last row; what
    // they produce lands in padding rows and is never used
    uint32_t vx[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int m = 8 * j + (lane >> 3);
        vx[j] = ((uint32_t)(gm0 + (m < rows ? m : rows - 1)) * (uint32_t)p.K + 8u * (uint32_t)(lane & 7)) * 2u;
    }
    // l1s: the B operand of down-projection step s (channels 32 lh + 8 s .. + 7) is the stored lane 16 (2 lh + s / 2) + l % 16 of k step
    // s % 2 and of the column's block of 16; columns past the rank are zeros
    int vl[RC];
#pragma unroll
    for (int c = 0; c < RC; ++c) {
        const int block = 2 * c + (li >> 4);
        vl[c] = block < rb ? block * 1024 + (32 * lh + (li & 15)) * 16 : kOff;
    }
    struct XSet { u32x4 x[4]; uint32_t r; };
    u32x4 lf[RC][4];
    auto load_x = [&](int g) {
        XSet s;
#pragma unroll
        for (int j = 0; j < 4; ++j) s.x[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, (int)vx[j], g * 128, 2));      // (streaming hint: X is read once)
        s.r = __builtin_amdgcn_raw_buffer_load_b32(rs_r, 4 * lane, g * 256, 0);
        return s;
    };
    auto load_l = [&](int g) {
#pragma unroll
        for (int c = 0; c < RC; ++c)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                lf[c][k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_l, vl[c] + 256 * (k / 2), (g * 2 + k % 2) * rb * 1024, 0));
    };
    floatx16 hacc[RC];
#pragma unroll
    for (int c = 0; c < RC; ++c) hacc[c] = floatx16{0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    unsigned char *xl = lds + wave * L::kWave;      // only this wavefront touches it: its LDS queue is in order, no barrier
    float *lrinv = reinterpret_cast<float *>(xl + 32 * kXRow);
    int g = gbeg + wave;
    XSet cur;
    if (g < gend) {
        cur = load_x(g);
        load_l(g);
    }
    for (; g < gend; g += WAVES) {
        const bool more = g + WAVES < gend;
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4 *>(xl + (8 * j + (lane >> 3)) * kXRow + 16 * (lane & 7)) = cur.x[j];
        reinterpret_cast<uint32_t *>(lrinv)[lane] = cur.r;
        if (more) cur = load_x(g + WAVES);
        u32x4 raw[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) raw[k] = *reinterpret_cast<const u32x4 *>(xl + li * kXRow + 64 * lh + 16 * k);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int c = 0; c < RC; ++c)
                hacc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, raw[k]), __builtin_bit_cast(bf16x8, lf[c][k]), hacc[c], 0, 0, 0);
        if (more) load_l(g + WAVES);
        float x[32], amax = 0.f;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const float4 r = *reinterpret_cast<const float4 *>(lrinv + 32 * lh + 4 * k);
            const uint32_t a = raw[k / 2][2 * (k & 1)], b = raw[k / 2][2 * (k & 1) + 1];
            x[4 * k] = bf16lo(a) * r.x;
            x[4 * k + 1] = bf16hi(a) * r.y;
            x[4 * k + 2] = bf16lo(b) * r.z;
            x[4 * k + 3] = bf16hi(b) * r.w;
        }
#pragma unroll
        for (int e = 0; e < 32; ++e) amax = fmaxf(amax, fabsf(x[e]));
        unsigned char *k = xl;      // (X has been read)
        if constexpr (FMT == 0) {
            const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(amax), __float_as_uint(amax), false, false);      // the token's other 32 channels
            uint32_t sx;
            const float rcp = w4_rcp_of(fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1])), sx);
            const act_u32x6 q = w4_codes32(x, rcp);
#pragma unroll
            for (int e = 0; e < 3; ++e) *reinterpret_cast<uint2 *>(k + 24 * lane + 8 * e) = make_uint2(q[2 * e], q[2 * e + 1]);
            if (lh == 0) *reinterpret_cast<uint32_t *>(k + kW4ACodes + 4 * lane) = sx;
            const buffer_u32x4 v0 = *reinterpret_cast<const buffer_u32x4 *>(k + 16 * lane), v1 = *reinterpret_cast<const buffer_u32x4 *>(k + 1024 + 16 * (lane < 40 ? lane : 0));
            const int sc = (g * (p.Mpad / 32) + gm0 / 32) * kW4ABlock;
            buffer_store_b128<0>(v0, rs_c, 16 * lane, sc);
            if (lane < 40) buffer_store_b128<0>(v1, rs_c, 1024 + 16 * lane, sc);
        } else {
            uint32_t sbyte;
            const uint4 q = fp4_encode32(x, amax, sbyte);
            buffer_store_b128<0>(__builtin_bit_cast(buffer_u32x4, q), rs_c, 16 * lane, (g * p.Mpad + gm0) * kFp4RowBytes);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)sbyte, rs_s, 4 * lane, ((g >> 2) * p.Mpad + gm0) * 8 + (g & 3), 0);
        }
    }
    // ---- the run's partial H: the wavefronts' parts meet in LDS, in their order (its codes have left in the loop)
    float *hmine = reinterpret_cast<float *>(xl);
#pragma unroll
    for (int c = 0; c < RC; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) hmine[(8 * (v >> 2) + 4 * lh + (v & 3)) * L::kHRow + 32 * c + li] = hacc[c][v];
    __syncthreads();
    for (int i = blockIdx.x * (WAVES * 64) + threadIdx.x; i < p.n_zero; i += gridDim.x * (WAVES * 64)) p.zero_words[i] = 0u;      // arrival counters of the GEMM that follows
    float *part = p.hpart + ((size_t)run * p.M + gm0) * p.rank;
    for (int idx = threadIdx.x; idx < rows * (p.rank / 4); idx += WAVES * 64) {
        const int r = idx / (p.rank / 4), col = 4 * (idx - r * (p.rank / 4));
        float4 h = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float4 t = *reinterpret_cast<const float4 *>(lds + w * L::kWave + (r * L::kHRow + col) * 4);
            h.x += t.x; h.y += t.y; h.z += t.z; h.w += t.w;
        }
        *reinterpret_cast<float4 *>(part + (size_t)r * p.rank + col) = h;
    }
}

template <int FMT, int RC>
hipError_t launch_tile(const ActParams &p, hipStream_t stream) {
    auto k = act_tile_kernel<FMT, RC>;
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), TileLds<RC>::kBytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)((p.M + kActTileTokens - 1) / kActTileTokens * p.chunks)), dim3(WAVES * 64), TileLds<RC>::kBytes, stream, p);
    return hipGetLastError();
}

template <int FMT>
hipError_t launch_rank(const ActParams &p, hipStream_t stream) {
    return p.rank <= 32 ? launch_tile<FMT, 1>(p, stream) : p.rank <= 64 ? launch_tile<FMT, 2>(p, stream) : launch_tile<FMT, 4>(p, stream);
}

}  // namespace

hipError_t launch_act_tile(const ActParams &p, hipStream_t stream) {
    if (p.M <= 0) return hipSuccess;
    if ((p.fmt != 0 && p.fmt != 1) || p.K != p.G * kGroup || p.rank <= 0 || p.rank > 128 || p.rank % 16 || p.Mpad % kRowPad || p.Mpad < p.M || (p.fmt == 1 && !p.sx) || !p.hpart ||
        p.chunks < 1 || p.gchunk < 1 || (size_t)p.gchunk * p.chunks < (size_t)p.G || (p.chunks - 1) * p.gchunk >= p.G || (size_t)p.K * p.Mpad >= ((size_t)1 << 31))
        return hipErrorInvalidValue;
    return p.fmt == 0 ? launch_rank<0>(p, stream) : launch_rank<1>(p, stream);
}

}  // namespace svdq
