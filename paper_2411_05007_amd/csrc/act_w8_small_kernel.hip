// The 8-bit setting's activation kernel for small batches (arXiv 2411.05007 App. "Implementation Details": per-token dynamic INT8;
// Sec. 4.3: quantization and down projection share their input): one launch, two kinds of workgroups.
//
// A token's scale needs its maximum over all of K before the first code can be written.  With 16 tokens to a workgroup, as
// the projection's matrix instruction wants them, a small batch is a handful of workgroups that each pull all of K and all L1
// fragments through one CU (12 us at one token, K = 6080), and cutting K takes a launch of its own for the maxima.  Here the first workgroups
// quantize, four tokens each: sixteen wavefronts hold the tokens' whole K in registers, wavefront w the 128-channel units w, w +
// 16, ...; the others project, 16 tokens and a run of K each, and leave the run's partial H for the GEMM to add.  Neither
// waits for the other.  Bound: one round trip for X and the smoothing factors (or X and the L1 fragments), a barrier, the
// stores.  us in a kernel trace: one pass 12.4 (M = 2, K = 6080, rank 16), two launches over a cut K 4.0 + 11.1 (M = 5, K = 8960, rank 32);
// this kernel 3.0 (M = 3, K = 1664), 4.0 (M = 16, K = 4864, ranks 16 and 32).  Which calls take it: layout.h, act_w8_small.
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
constexpr int kWaves = 16, kTokens = 4;

// RB: rank / 16 (0: no projection; the GEMM that adds the runs takes two rank steps at most); UN: units of 128 channels per quantizing wavefront
template <int RB, int UN>
__global__ __launch_bounds__(kWaves * 64, 1) void act_w8_small_kernel(ActParams p, int quantizers) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // housekeeping for the kernel that follows on the stream: its tile arrival counters start at zero
    for (int i = blockIdx.x * (kWaves * 64) + threadIdx.x; i < p.n_zero; i += gridDim.x * (kWaves * 64)) p.zero_words[i] = 0u;
    if ((int)blockIdx.x < quantizers) {
        // lane l: token l / 16, channels 8 (l % 16) .. + 7 of a unit; rows past M read the last row, their codes land in padding rows
        const int c16 = lane & 15, m = blockIdx.x * kTokens + (lane >> 4);
        const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.X, (size_t)p.M * p.K * 2);
        const __amdgpu_buffer_rsrc_t rs_r = make_rsrc(p.rinv, (size_t)p.K * 4);
        const __amdgpu_buffer_rsrc_t rs_c = make_rsrc(p.codes, (size_t)p.K * p.Mpad);
        // (byte offsets below 2^32: the entry point refuses batches of 2^31 elements or more; unsigned on purpose)
        const uint32_t vx = ((uint32_t)(m < p.M ? m : p.M - 1) * (uint32_t)p.K + 8u * (uint32_t)c16) * 2u;
        const int vc = (int)i8_code_offset(8 * c16, p.Mpad, m);
        auto unit = [&](int i) { return wave + kWaves * i; };
        auto live = [&](int i) { return 128 * unit(i) + 8 * c16 < p.K; };      // the lane's channels exist (an odd number of groups: half a unit)
        uint4 x[UN];
        float4 r0[UN], r1[UN];
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            x[i] = make_uint4(0u, 0u, 0u, 0u);
            r0[i] = r1[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (live(i)) {
                x[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, (int)vx, unit(i) * 256, 0));
                r0[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs_r, 32 * c16, unit(i) * 512, 0));
                r1[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rs_r, 32 * c16 + 16, unit(i) * 512, 0));
            }
        }
        auto smooth = [&](int i, float (&o)[8]) {
            const uint32_t w[4] = {x[i].x, x[i].y, x[i].z, x[i].w};
            const float r[8] = {r0[i].x, r0[i].y, r0[i].z, r0[i].w, r1[i].x, r1[i].y, r1[i].z, r1[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                o[2 * e] = bf16lo(w[e]) * r[2 * e];
                o[2 * e + 1] = bf16hi(w[e]) * r[2 * e + 1];
            }
        };
        float amax = 0.f;
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            float t[8];
            smooth(i, t);
#pragma unroll
            for (int e = 0; e < 8; ++e) amax = fmaxf(amax, fabsf(t[e]));
        }
        amax = max_over_8_lanes(amax);
        amax = fmaxf(amax, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, amax), 0x140, 0xf, 0xf, true)));      // row_mirror: the token's other eight lanes
        float *mx = reinterpret_cast<float *>(lds);      // [4 tokens][wavefronts]
        if (c16 == 0) mx[(lane >> 4) * kWaves + wave] = amax;
        __syncthreads();
        const float4 *q = reinterpret_cast<const float4 *>(mx + (lane >> 4) * kWaves);
        amax = 0.f;
#pragma unroll
        for (int k = 0; k < kWaves / 4; ++k) amax = fmaxf(fmaxf(amax, fmaxf(q[k].x, q[k].y)), fmaxf(q[k].z, q[k].w));
        // Eq. 1 with q_max = 127: s = fp16(max / 127) (IEEE division, round to nearest even, saturating), codes from x^ * (1.0f / s)
        float s32 = amax / 127.0f;
        s32 = fminf(s32, 65504.0f);
        const _Float16 sh = (_Float16)s32;
        const float sc = (float)sh;
        const float rcp = sc > 0.f ? 1.0f / sc : 0.f;
        if (wave == 0 && c16 == 0) p.sx[m] = __builtin_bit_cast(uint16_t, sh);      // < Mpad
#pragma unroll
        for (int i = 0; i < UN; ++i) {
            float t[8];
            smooth(i, t);
            uint32_t w[2] = {0u, 0u};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float c = fminf(127.f, fmaxf(-127.f, __builtin_rintf(t[e] * rcp)));
                w[e >> 2] |= ((uint32_t)(int)c & 0xffu) << (8 * (e & 3));
            }
            if (live(i)) __builtin_amdgcn_raw_buffer_store_b64(u32x2{w[0], w[1]}, rs_c, vc, unit(i) * 128 * p.Mpad, 0);      // a unit is four 32-channel steps of operand blocks
        }
    } else if constexpr (RB > 0) {
        const int job = (int)blockIdx.x - quantizers, slice = job / p.chunks, chunk = job - slice * p.chunks;
        const int row = lane & 15, blk = lane >> 4, m0 = slice * 16, rb = p.rank / 16;
        const int gbeg = chunk * p.gchunk, gend = gbeg + p.gchunk < p.G ? gbeg + p.gchunk : p.G;
        const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.X, (size_t)p.M * p.K * 2);
        const __amdgpu_buffer_rsrc_t rs_l = make_rsrc(p.l1s, (size_t)p.K * p.rank * 2);
        const uint32_t vx = ((uint32_t)(m0 + row < p.M ? m0 + row : p.M - 1) * (uint32_t)p.K + 16u * (uint32_t)blk) * 2u;
        floatx4 acc[RB];
#pragma unroll
        for (int c = 0; c < RB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
        struct Set { uint4 x[2], b[2 * RB]; };
        auto load = [&](Set &s, int g) {
#pragma unroll
            for (int k = 0; k < 2; ++k) s.x[k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, (int)vx + 16 * k, g * 128, 0));
#pragma unroll
            for (int c = 0; c < RB; ++c) {
                const int cc = c < rb ? c : rb - 1;      // blocks past the rank repeat the last one; their sums are dropped
                s.b[2 * c] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_l, lane * 16, (g * 2 * rb + cc) * 1024, 0));
                s.b[2 * c + 1] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs_l, lane * 16, ((g * 2 + 1) * rb + cc) * 1024, 0));
            }
        };
        auto multiply = [&](const Set &s) {
#pragma unroll
            for (int c = 0; c < RB; ++c)
#pragma unroll
                for (int k = 0; k < 2; ++k)
                    acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, s.x[k]), __builtin_bit_cast(bf16x8, s.b[2 * c + k]), acc[c], 0, 0, 0);
        };
        constexpr int kSets = 2;      // groups requested together
        for (int g = gbeg + wave; g < gend; g += kSets * kWaves) {
            Set s[kSets];
            load(s[0], g);
            if (g + kWaves < gend) load(s[kSets - 1], g + kWaves);
            __builtin_amdgcn_sched_barrier(0);
            multiply(s[0]);
            if (g + kWaves < gend) multiply(s[kSets - 1]);
        }
        // the wavefronts' sums, added in wavefront order
        constexpr int kRow = 16 * RB + 1;
        float *red = reinterpret_cast<float *>(lds);      // [wave][16 tokens][kRow]
#pragma unroll
        for (int c = 0; c < RB; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[(wave * 16 + 4 * blk + v) * kRow + 16 * c + row] = acc[c][v];
        __syncthreads();
        if (job == 0 && threadIdx.x == 0) h_in_parts(p.H, p.hpart, p.chunks);
        float *mine = p.hpart + ((size_t)chunk * p.Mpad + m0) * p.rank;
        for (int idx = threadIdx.x; idx < 16 * p.rank; idx += kWaves * 64) {
            const int r = idx / p.rank, col = idx - r * p.rank;
            float h = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) h += red[(w * 16 + r) * kRow + col];
            mine[idx] = h;
        }
    }
}

template <int RB, int UN>
hipError_t launch_small(const ActParams &p, hipStream_t stream) {
    auto k = act_w8_small_kernel<RB, UN>;
    constexpr int bytes = RB > 0 ? kWaves * 16 * (16 * RB + 1) * 4 : kTokens * kWaves * 4;
    static_assert(bytes <= kLdsBytesPerCU && bytes >= kTokens * kWaves * 4, "");
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), bytes); e != hipSuccess) return e;
    const int quantizers = (p.M + kTokens - 1) / kTokens, projectors = RB > 0 ? (p.M + 15) / 16 * p.chunks : 0;
    hipLaunchKernelGGL(k, dim3((unsigned)(quantizers + projectors)), dim3(kWaves * 64), bytes, stream, p, quantizers);
    return hipGetLastError();
}
template <int RB>
hipError_t launch_units(const ActParams &p, hipStream_t stream) {
    const int units = (p.G + 1) / 2;
    if (units <= kWaves) return launch_small<RB, 1>(p, stream);
    if (units <= 2 * kWaves) return launch_small<RB, 2>(p, stream);
    if (units <= 3 * kWaves) return launch_small<RB, 3>(p, stream);
    return launch_small<RB, 6>(p, stream);
}

}  // namespace

hipError_t launch_act_w8_small(const ActParams &p, int flags, hipStream_t stream) {
    if (p.M <= 0) return hipSuccess;
    const int rank = (flags & 2) ? p.rank : 0;
    if (p.fmt != 2 || !(flags & 1) || !p.sx || p.K != p.G * kGroup || p.G > kActW8SmallGroups || rank > 32 || p.rank % 16 || (size_t)p.K * p.Mpad >= ((size_t)1 << 31) ||
        p.Mpad % kRowPad || p.Mpad < p.M)
        return hipErrorInvalidValue;
    if (rank > 0 && (!p.hpart || p.chunks < 1 || (size_t)p.gchunk * p.chunks < (size_t)p.G || (p.chunks - 1) * p.gchunk >= p.G)) return hipErrorInvalidValue;      // runs that cover K, none empty
    if (rank == 0) return launch_units<0>(p, stream);
    return rank <= 16 ? launch_units<1>(p, stream) : launch_units<2>(p, stream);
}

}  // namespace svdq
