// The whole forward of a small batch in ONE launch (arXiv 2411.05007 Eq. 5, Sec. 4.3): smoothing, quantization, down projection,
// 4-bit product, up projection and bias, for INT4 and MXFP4 layers.
//
// A forward of few tokens is two short kernels of a few round trips each: two launches that do nothing follow each other every 5.7 us
// here, one every 2.8, and the second kernel starts cold behind the first.  Here every workgroup quantizes the 32 tokens of its
// tile by itself, as many times over as the launch has tiles side by side, and waits for nobody.  Bound: what that costs a CU per group of
// K, 225 vector instructions of a wavefront (four clocks each, 170 of them the quantizer's) and ten kilobytes through its load path (X and
// l1s four each), which add up to 0.13 us; with a start of 1.2 us, a first step as long and 1.6 us for the meeting, the low-rank product
// and the stores (time stamps inside the kernel).  So it is for short K and narrow branches: us per forward, two launches -> this,
// M = 256, K = N = 1152, rank 32: INT4 9.2 -> 7.2, MXFP4 9.0 -> 6.9; the rule, with both sides: layout.h, fused_small.
// Tried: sixteen wavefronts (K = 1152 7.9, K = 3072 11.5 us, two launches 10.3: the vector instructions are what it takes, not their latency),
// the quantizer in X's load map (eight lanes to a token: a reciprocal for every eighth of the tokens, 360 instructions).
//
// A workgroup owns a 32 x 64 tile and its eight wavefronts share K, wavefront w taking groups w, w + 8, ..., as in
// gemm_w4a4_kpar_kernel.hip.  A wavefront reads X of a group in whole 128-byte lines and turns it through its own block of LDS
// into the operand map of the matrix instructions (lane l: token l % 32, channels 32 (l / 32) .. + 31 of the group), in which
// everything else happens without another exchange: the raw values are the A operand of the down projection
// (v_mfma_f32_32x32x16_bf16 against l1s, four steps of 8 channels per lane half), a lane's 32 smoothed channels are half of an INT4
// group (one permlane for its maximum) or a whole MXFP4 block, and the conversion instructions return the codes as the
// operand registers of the 4-bit product.  Behind the loop the wavefronts' partial H and partial tiles meet in LDS; every
// wavefront adds up eight rows of one column block, and the up projection is added to them by the same bf16 instructions on H's hi
// and lo parts.
// The workspace gets what the two-launch forward leaves in it (activation blocks and H, which svdq_debug_act reads): a tile's
// workgroup keeps the codes of its share of the groups in LDS and stores them behind the loop, where no load waits behind a store.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "act_common.h"
#include "buffer.h"
#include "gemm_kpar.h"
#include "kernels.h"
#include "layout.h"
#include "lds_limit.h"

namespace svdq {
namespace {

typedef int intx8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 halfx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 8, kDepth = 2;          // wavefronts, and groups whose operands a wavefront asks for ahead
constexpr int kFmtE2M3 = 2, kFmtE2M1 = 4;     // operand format selectors of the block-scaled instruction
constexpr int kScaleBytes = 0x8082;           // INT4: block scales 2^3 and 2^1, as in gemm_w4a4_kernel.hip
constexpr int kXRow = 144;                    // 128 bytes of a token's group + 16: the 32 rows of an operand read fall on distinct banks
constexpr int kOff = (int)0x80000000u;        // a lane offset beyond every buffer (layout.h, kpar_step): the load returns zeros

// LDS: the wavefronts' partial tiles, in whose places X is turned around and 1 / lambda of a group lies before; the store blocks of
// gemm_kpar.h; the wavefronts' partial H; H's bf16 parts; the codes that the workgroup will store.
using Tile = KparLds<1, 2, kWaves>;
constexpr int kTileBytes = 8192;
static_assert(Tile::kPart == kWaves * kTileBytes && 32 * kXRow + 256 <= kTileBytes, "");
constexpr int kRank = 32;                      // columns of H, zeros past the rank
template <int FMT, bool LOWRANK> struct FusedLds {
    static constexpr int kCodeBytes = FMT == 0 ? kW4AUsed : 1024 + 64;
    static constexpr int kHRow = kRank + 8;      // words; the two lane halves' rows, four apart, fall on different banks
    static constexpr int kHpart = Tile::kBytes, kHsum = kHpart + (LOWRANK ? kWaves * 32 * kHRow * 4 : 0), kKeep = kHsum + (LOWRANK ? 32 * kRank * 4 : 0);
};

// FMT 0: INT4, 1: MXFP4.  LOWRANK: the layer has a 16-bit branch
template <int FMT, bool LOWRANK>
__global__ __launch_bounds__(kWaves * 64, 1) void fused_small_kernel(FusedSmallParams p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    using L = FusedLds<FMT, LOWRANK>;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lh = lane >> 5;      // operand map: row or column li, channels 32 lh .. + 31 of the group
    const int tiles_m = (p.M + 31) / 32, tiles_n = (p.N + 63) / 64;
    int tile_m, tile_n;
    kpar_tile_of((int)blockIdx.x, tiles_m, tiles_n, 128, FMT == 0 ? kW4BBlock / 64 : 34, tile_m, tile_n);
    const int gm0 = tile_m * 32, gn0 = tile_n * 64;      // the launch checks that every tile lies inside the padded rows and columns
    const int rows = p.M - gm0 < 32 ? p.M - gm0 : 32;
    const int rb = p.rank / 16;

    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.X, (size_t)p.M * p.K * 2);
    const __amdgpu_buffer_rsrc_t rs_r = make_rsrc(p.rinv, (size_t)p.K * 4);
    const __amdgpu_buffer_rsrc_t rs_l = make_rsrc(p.l1s, (size_t)p.K * p.rank * 2);
    const __amdgpu_buffer_rsrc_t rs_w = make_rsrc(p.wcodes, FMT == 0 ? w4_b_bytes(p.G, p.Npad) : (size_t)p.G * p.Npad * kFp4RowBytes);
    const __amdgpu_buffer_rsrc_t rs_s = make_rsrc(p.bw, FMT == 0 ? 0 : fp4_scale_bytes(p.G, p.Npad));

    // ---- requests: a wavefront's operands of one group, kDepth groups ahead; past the end of K nothing
    struct Set { u32x4 x[4], w[2], l[4]; uint32_t s[2], r; };
    Set S[kDepth];
    // load map of X: request j reads tokens 8 j + lane / 8, channels 8 (lane % 8) .. + 7 of the group; tokens past M are zeros
    auto load_x = [&](Set &s, int g) {
        const int past = g < p.G ? 0 : kOff, gc = g < p.G ? g : 0, row = lane >> 3;
        const int v = (int)(((uint32_t)(gm0 + row) * (uint32_t)p.K + 8u * (uint32_t)(lane & 7)) * 2u);
#pragma unroll
        for (int j = 0; j < 4; ++j) s.x[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, (8 * j + row < rows ? v + j * 16 * p.K : kOff) | past, gc * 128, 0));
        s.r = __builtin_amdgcn_raw_buffer_load_b32(rs_r, (4 * lane) | past, gc * 256, 0);
    };
    // l1s: the B operand of down-projection step s (channels 32 lh + 8 s .. + 7) is the stored lane 16 (2 lh + s / 2) + l % 16 of k step
    // s % 2 and of the column's block of 16; columns past the rank are zeros
    auto load_l = [&](Set &s, int g) {
        const int past = g < p.G ? 0 : kOff, gc = g < p.G ? g : 0, block = li >> 4;
        const int v = (block < rb ? block * 1024 + (32 * lh + (lane & 15)) * 16 : kOff) | past;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (LOWRANK) s.l[k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_l, v + 256 * (k / 2), (gc * 2 + k % 2) * rb * 1024, 0));
    };
    auto load_w = [&](Set &s, int g) {
        const int past = g < p.G ? 0 : kOff, gc = g < p.G ? g : 0;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (FMT == 0) {
                const int at = (gc * (p.Npad / 64) + gn0 / 64) * kW4BBlock;
                s.w[c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_w, (16 * lane) | past, at + c * 1024, 0));
                s.s[c] = __builtin_amdgcn_raw_buffer_load_b32(rs_w, (kW4BCodes + 4 * li) | past, at + c * 128, 0);
            } else {
                s.w[c] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_w, (16 * lane) | past, (gc * p.Npad + gn0) * kFp4RowBytes + c * 1024, 0));
                s.s[c] = __builtin_amdgcn_raw_buffer_load_b32(rs_s, (4 * lane) | past, ((gc >> 2) * p.Npad + gn0) * 8 + c * 256, 0);
            }
        }
    };
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
        load_x(S[d], wave + kWaves * d);
        load_l(S[d], wave + kWaves * d);
        load_w(S[d], wave + kWaves * d);
        __builtin_amdgcn_sched_barrier(0);
    }
    // what the wavefront finishes: rows 8 oct .. + 7 of column block cb
    const int oct = wave >> 1, cb = wave & 1, col = gn0 + 32 * cb + li;      // < Npad
    const float bias = p.bias[col];
    u32x4 l2[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) l2[ks] = LOWRANK && ks < rb ? __builtin_bit_cast(u32x4, *reinterpret_cast<const uint4 *>(p.l2t + (size_t)col * p.rank + 16 * ks + 8 * lh)) : u32x4{0u, 0u, 0u, 0u};

    // the groups whose codes this workgroup stores
    const int own = (p.G + tiles_n - 1) / tiles_n, own0 = tile_n * own;
    unsigned char *keep = lds + L::kKeep;

    // ---- the loop ------------------------------------------------------------------------------------------------
    const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    floatx16 acc4[2] = {zero16, zero16}, hacc = zero16;      // (MXFP4: the instruction adds up by itself)
    float acc[2][16];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[c][v] = 0.f;
    int scales = kScaleBytes;
    asm volatile("" : "+v"(scales));
    unsigned char *xl = lds + wave * kTileBytes;      // only this wavefront touches it: its LDS queue is in order, no barrier
    float *lrinv = reinterpret_cast<float *>(xl + 32 * kXRow);
    auto step = [&](Set &s, int g) {
        // X through LDS into the operand map, and its down projection
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<u32x4 *>(xl + (8 * j + (lane >> 3)) * kXRow + 16 * (lane & 7)) = s.x[j];
        reinterpret_cast<uint32_t *>(lrinv)[lane] = s.r;
        if (g + kDepth * kWaves < p.G) load_x(s, g + kDepth * kWaves);
        u32x4 raw[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) raw[k] = *reinterpret_cast<const u32x4 *>(xl + li * kXRow + 64 * lh + 16 * k);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (LOWRANK) hacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, raw[k]), __builtin_bit_cast(bf16x8, s.l[k]), hacc, 0, 0, 0);
        if (g + kDepth * kWaves < p.G) load_l(s, g + kDepth * kWaves);
        // the lane's 32 smoothed channels and their codes
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
        unsigned char *k = keep + (g - own0) * L::kCodeBytes;
        const bool mine = (unsigned)(g - own0) < (unsigned)own;
        if constexpr (FMT == 0) {
            const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(amax), __float_as_uint(amax), false, false);      // the token's other 32 channels
            uint32_t sx;
            const float rcp = w4_rcp_of(fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1])), sx);
            const act_u32x6 q = w4_codes32(x, rcp);
            if (mine) {
#pragma unroll
                for (int e = 0; e < 3; ++e) *reinterpret_cast<uint2 *>(k + 24 * lane + 8 * e) = make_uint2(q[2 * e], q[2 * e + 1]);
                if (lh == 0) *reinterpret_cast<uint32_t *>(k + kW4ACodes + 4 * lane) = sx;
            }
            const intx8 a = {(int)q[0], (int)q[1], (int)q[2], (int)q[3], (int)q[4], (int)q[5], 0, 0};
            struct Pair { uint32_t lo, hi; };
            const halfx4 sa = __builtin_bit_cast(halfx4, Pair{sx, sx});
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const u32x4 w = s.w[c];
                const intx8 b = {(int)(w.x & ~kW4Z0), (int)(w.y & ~kW4Z1), (int)((w.x & kW4Z0) | (w.y & kW4Z1)),
                                 (int)(w.z & ~kW4Z0), (int)(w.w & ~kW4Z1), (int)((w.z & kW4Z0) | (w.w & kW4Z1)), 0, 0};
                const floatx16 ag = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, zero16, kFmtE2M3, kFmtE2M3, 0, scales, 1, scales);
                const floatx16 sg = __builtin_amdgcn_mfma_f32_32x32x8f16(sa, __builtin_bit_cast(halfx4, Pair{s.s[c], s.s[c]}), zero16, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[c][v] = __builtin_fmaf(ag[v], sg[v], acc[c][v]);
            }
        } else {
            uint32_t sbyte;
            const uint4 q = fp4_encode32(x, amax, sbyte);
            if (mine) {
                *reinterpret_cast<uint4 *>(k + 16 * lane) = q;
                k[1024 + lane] = (unsigned char)sbyte;
            }
            const intx8 a = {(int)q.x, (int)q.y, (int)q.z, (int)q.w, 0, 0, 0, 0};
            const int shift = (wave & 3) * 8;      // the wavefront's place in every chunk of four groups
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const intx8 b = {(int)s.w[c].x, (int)s.w[c].y, (int)s.w[c].z, (int)s.w[c].w, 0, 0, 0, 0};
                acc4[c] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc4[c], kFmtE2M1, kFmtE2M1, 0, (int)sbyte, 0, (int)(s.s[c] >> shift));
            }
        }
        if (g + kDepth * kWaves < p.G) load_w(s, g + kDepth * kWaves);
    };
    for (int g = wave; g < p.G; g += kDepth * kWaves)
#pragma unroll
        for (int d = 0; d < kDepth; ++d) {
            if (d > 0 && g + d * kWaves >= p.G) break;
            step(S[d], g + d * kWaves);
        }
    if constexpr (FMT == 1)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[c][v] = acc4[c][v];

    // ---- the wavefronts meet -------------------------------------------------------------------------------------
    float *hpart = reinterpret_cast<float *>(lds + L::kHpart);
#pragma unroll
    for (int v = 0; v < 16; ++v)
        if (LOWRANK) hpart[(wave * 32 + 8 * (v >> 2) + 4 * lh + (v & 3)) * L::kHRow + li] = hacc[v];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int c = 0; c < 2; ++c) *reinterpret_cast<float4 *>(xl + (q * 2 + c) * 1024 + lane * 16) = make_float4(acc[c][4 * q], acc[c][4 * q + 1], acc[c][4 * q + 2], acc[c][4 * q + 3]);
    __syncthreads();
    Kpar4<float> sum{};
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const float4 t = *reinterpret_cast<const float4 *>(lds + w * kTileBytes + (oct * 2 + cb) * 1024 + lane * 16);
        sum.x += t.x; sum.y += t.y; sum.z += t.z; sum.w += t.w;
    }
    if constexpr (LOWRANK) {
        // H: two columns of a token per thread, the partial H in their order, into the bf16 parts
        const int half = p.rank / 2;
        for (int idx = threadIdx.x; idx < 32 * half; idx += kWaves * 64) {
            const int row = idx / half, j = 2 * (idx - row * half);
            float h0 = 0.f, h1 = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const float2 t = *reinterpret_cast<const float2 *>(hpart + (w * 32 + row) * L::kHRow + j);
                h0 += t.x;
                h1 += t.y;
            }
            const uint32_t hi = bf16_rne_pair(h0, h1), lo = bf16_rne_pair(h0 - bf16lo(hi), h1 - bf16hi(hi));
            unsigned char *o = lds + L::kHsum + 2 * (j & 7);
            *reinterpret_cast<uint32_t *>(o + hfrag_offset(p.rank, row, j, 0)) = hi;
            *reinterpret_cast<uint32_t *>(o + hfrag_offset(p.rank, row, j, 1)) = lo;
            if (tile_n == 0) *reinterpret_cast<float2 *>(p.H + (size_t)(gm0 + row) * p.rank + j) = make_float2(h0, h1);      // row < Mpad
        }
        __syncthreads();
        floatx16 y;
#pragma unroll
        for (int q = 0; q < 4; ++q) { y[4 * q] = sum.x; y[4 * q + 1] = sum.y; y[4 * q + 2] = sum.z; y[4 * q + 3] = sum.w; }      // quad `oct` counts
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            if (ks < rb) {
                const unsigned char *h = lds + L::kHsum + ks * 2048 + lane * 16;
                y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(h)), __builtin_bit_cast(bf16x8, l2[ks]), y, 0, 0, 0);
                y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(h + 1024)), __builtin_bit_cast(bf16x8, l2[ks]), y, 0, 0, 0);
            }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (oct == q) sum = Kpar4<float>{y[4 * q], y[4 * q + 1], y[4 * q + 2], y[4 * q + 3]};
    }
    KparStore<1, 2, kWaves> out(lds, wave, lane);
    out.put(0, 0, Kpar4<float>{sum.x + bias, sum.y + bias, sum.z + bias, sum.w + bias});
    out.store(0, p.Y, p.M, p.N, gm0, gn0);

    // the activation blocks of this workgroup's groups
    const int have = p.G - own0 < own ? p.G - own0 : own;      // (negative: none)
    if constexpr (FMT == 0) {
        constexpr int kChunks = kW4AUsed / 16;
        for (int idx = threadIdx.x; idx < have * kChunks; idx += kWaves * 64) {
            const int k = idx / kChunks, at = 16 * (idx - k * kChunks);
            *reinterpret_cast<uint4 *>(p.codes + w4_a_block(own0 + k, p.Mpad, gm0) + at) = *reinterpret_cast<const uint4 *>(keep + k * L::kCodeBytes + at);
        }
    } else {
        for (int k = wave; k < have; k += kWaves) {
            *reinterpret_cast<uint4 *>(p.codes + fp4_code_offset(own0 + k, p.Mpad, gm0, 0) + 16 * lane) = *reinterpret_cast<const uint4 *>(keep + k * L::kCodeBytes + 16 * lane);
            p.bx[fp4_scale_offset(own0 + k, p.Mpad, gm0 + li, lh)] = keep[k * L::kCodeBytes + 1024 + lane];
        }
    }
}

template <int FMT, bool LOWRANK>
hipError_t launch_one(const FusedSmallParams &p, hipStream_t stream) {
    using L = FusedLds<FMT, LOWRANK>;
    const int tiles_m = (p.M + 31) / 32, tiles_n = (p.N + 63) / 64, own = (p.G + tiles_n - 1) / tiles_n;
    if (L::kKeep + own * L::kCodeBytes > kLdsBytesPerCU) return hipErrorInvalidValue;
    auto k = fused_small_kernel<FMT, LOWRANK>;
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), kLdsBytesPerCU); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(tiles_m * tiles_n), dim3(kWaves * 64), L::kKeep + own * L::kCodeBytes, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fused_small(const FusedSmallParams &p, int fmt, hipStream_t stream) {
    if (p.M <= 0) return hipSuccess;
    // what the kernel's addressing assumes: whole tiles inside the padded rows and columns
    if (p.G <= 0 || p.K != p.G * kGroup || p.Mpad % kRowPad || p.Npad % kRowPad || p.Mpad < p.M || p.Npad < p.N || p.N % 16 || p.rank < 0 || p.rank % 16 || p.rank > kRank ||
        (p.rank > 0 && (!p.l1s || !p.l2t || !p.H)) || (fmt != 0 && fmt != 1))
        return hipErrorInvalidValue;
    if (fmt == 0) return p.rank > 0 ? launch_one<0, true>(p, stream) : launch_one<0, false>(p, stream);
    return p.rank > 0 ? launch_one<1, true>(p, stream) : launch_one<1, false>(p, stream);
}

}  // namespace svdq
