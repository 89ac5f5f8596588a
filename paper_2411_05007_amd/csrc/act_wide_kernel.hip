// Activation kernel for wide 16-bit branches (ranks 65 to 128) on batches that fill the chip: the arithmetic of act_kernel.hip
// (arXiv 2411.05007 Sec. 4.3, Fig. 6b: "Quantize" and "Down Projection" share their input; Eq. 1 per group), 64 tokens to a
// workgroup instead of 16.
//
// At rank 128 a group of 64 channels is 2 KB of X per 16 tokens and 16 KB of L1 fragments, and a launch of 16-token workgroups is
// bound by what the L2 delivers of the latter (M = 4608, K = 12288: 906 MB of 1045 in 70 us, 15 TB/s).  Here four wavefronts, 16
// tokens each, read one copy of the fragments: X, the fragments and 1 / lambda of a group go from memory into a three-stage LDS
// ring with direct-to-LDS loads, three groups ahead, one barrier per group.  A lane asks for the 16-byte chunk of a token's 128
// bytes that belongs at its place of a row whose chunks are permuted by the token's number, so that both the reads by token (codes)
// and those by the matrix instruction's operand map fall on distinct banks.  K is cut into runs; a workgroup leaves its partial H in
// scratch memory with plain stores, and a small launch of its own (act_sum_h) adds the runs in order: every wavefront owns its
// tokens, nothing meets here.
// us in a kernel trace at M = 4608, K = 12288, rank 128: act_kernel.hip 74.5; this kernel 52 and the sum 5.7 (504 workgroups; 576, which is a
// second round, 67 + 6).  Bound: a group's chain in a workgroup (LDS reads, products, quantizer, barrier; 1.1 us alone, 1.8 with a second workgroup on
// the CU): timing-only copies that always hit the L2 with X or with the fragments, or that do not store codes, run at the same speed, one without the
// quantizer 6 us faster; asking LDS for the next group's operands in front of the quantizer changed nothing.
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
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void *lds_ptr;

constexpr int RB = 8;      // 16-column blocks of H (p.rank / 16 of them used)
template <int FMT>
struct WideLds {
    static constexpr int kX = kActWideTokens * 128, kL1 = RB * 2048, kRinv = 1024;      // (1 / lambda: 256 bytes, and the rest of one request)
    static constexpr int kStage = kX + kL1 + kRinv, kStages = 3;
    static constexpr int kOut = FMT == 0 ? 4 * kActOutStage + 256 : 0;                  // (a staged read is a whole wavefront's)
    static constexpr int kBytes = kStages * kStage + kOut;
    static constexpr int kReq = 2 + RB / 2 + 1;                                         // direct-to-LDS requests per wavefront and group
    static constexpr int kStores = FMT == 0 ? 1 : 3;                                    // code stores per wavefront and group
    static_assert(2 * kBytes <= kLdsBytesPerCU, "");
};

// FMT 0: INT4, 1: MXFP4
template <int FMT>
__global__ __launch_bounds__(256, 2) void act_wide_kernel(ActParams p) {
#ifdef __HIP_DEVICE_COMPILE__      // (as in gemm_w4a4_mid_kernel.hip)
    using L = WideLds<FMT>;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = lane & 15, blk = lane >> 4;      // MFMA operand / accumulator map
    const int r8 = lane >> 3, c8 = lane & 7;         // token map: tokens r8 and r8 + 8, channels 8 c8 .. + 7
    const int tile = (int)blockIdx.x / p.chunks, run = (int)blockIdx.x - tile * p.chunks;
    const int m0 = tile * kActWideTokens + 16 * wave, rb = p.rank / 16;
    const int gbeg = run * p.gchunk, gend = gbeg + p.gchunk < p.G ? gbeg + p.gchunk : p.G;

    // rows past M read the last row; what they produce lands in padding rows and is never used
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.X, (size_t)p.M * p.K * 2);
    const __amdgpu_buffer_rsrc_t rs_r = make_rsrc(p.rinv, (size_t)p.K * 4);
    const __amdgpu_buffer_rsrc_t rs_l = make_rsrc(p.l1s, (size_t)p.K * p.rank * 2);
    const __amdgpu_buffer_rsrc_t rs_c = make_rsrc(p.codes, FMT == 1 ? (size_t)p.G * p.Mpad * kFp4RowBytes : w4_a_bytes(p.G, p.Mpad));
    const __amdgpu_buffer_rsrc_t rs_s = make_rsrc(p.sx, FMT == 1 ? fp4_scale_bytes(p.G, p.Mpad) : 0);
    constexpr int kNowhere = (int)0x80000000u;      // a lane offset beyond every buffer that is addressed with it (all smaller than 2^31 bytes)
    // (byte offsets of X below 2^32: the entry point refuses batches of 2^31 elements or more; a lane that is to load nothing is given one past X)
    uint32_t vx[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int m = m0 + 8 * i + r8;
        vx[i] = ((uint32_t)(m < p.M ? m : p.M - 1) * (uint32_t)p.K + 8u * (uint32_t)(c8 ^ r8)) * 2u;
    }
    const int vr = lane < 16 ? 16 * lane : kNowhere;
    auto request = [&](int g, int stage) {
        // past the run's end: the last group once more, into a stage that is not read again, so that every step issues as many requests
        const int gc = g < gend ? g : gend - 1;
        unsigned char *st = lds + stage * L::kStage;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (lds_ptr)(st + (16 * wave + 8 * i) * 128), 16, (int)vx[i], gc * 128, 0, 2);      // (streaming hint: X is read once)
#pragma unroll
        for (int i = 0; i < RB / 2; ++i) {
            const int piece = wave + 4 * i;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_l, (lds_ptr)(st + L::kX + piece * 1024), 16, piece < 2 * rb ? lane * 16 : kNowhere, (gc * 2 * rb + (piece < 2 * rb ? piece : 0)) * 1024, 0, 0);
        }
        // (all four wavefronts bring the same 1 / lambda to the same place: as many requests for each)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_r, (lds_ptr)(st + L::kX + L::kL1), 16, vr, gc * 256, 0, 0);
    };

    // LDS traffic of the loop is written as instructions of its own, with explicit waits (the compiler would make every LDS access
    // wait for all outstanding memory-to-LDS requests); a wavefront's LDS operations complete in order
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    const uint32_t la_t = base + (16 * wave + r8) * 128 + 16 * (c8 ^ r8);                    // token r8; r8 + 8 lies 1024 bytes on
    const uint32_t la_m[2] = {base + (16 * wave + row) * 128 + 16 * ((2 * blk) ^ (row & 7)), base + (16 * wave + row) * 128 + 16 * ((2 * blk + 1) ^ (row & 7))};
    const uint32_t la_b = base + L::kX + 16 * lane, la_r = base + L::kX + L::kL1 + 32 * c8;
    const uint32_t la_out = base + L::kStages * L::kStage + wave * kActOutStage;
    const W4Stage w4(r8, c8);
    const int vout = w4_stage_out(m0, lane);
    const int ma = m0 + r8, mb = ma + 8;
    const int vca = (int)fp4_code_offset(0, p.Mpad, ma, c8 >> 2) + 4 * (c8 & 3), vcb = (int)fp4_code_offset(0, p.Mpad, mb, c8 >> 2) + 4 * (c8 & 3);
    const int vsx = (int)fp4_scale_offset(0, p.Mpad, (c8 & 1) ? mb : ma, c8 >> 2);
    floatx4 acc[RB];
#pragma unroll
    for (int c = 0; c < RB; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};

#define WIDE_READ(DST, ADDR, OFF) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(DST) : "v"(ADDR), "n"(OFF))
#define WIDE_WRITE(ADDR, VAL) asm volatile("ds_write_b32 %0, %1" ::"v"(ADDR), "v"(VAL) : "memory")
    u32x4 xa, xb, ra, rq, a0, a1, b[2 * RB];
    auto read = [&](int stage) {
        const uint32_t so = stage * L::kStage, at = la_t + so, am0 = la_m[0] + so, am1 = la_m[1] + so, ab = la_b + so, ar = la_r + so;
        WIDE_READ(xa, at, 0);
        WIDE_READ(xb, at, 1024);
        WIDE_READ(ra, ar, 0);
        WIDE_READ(rq, ar, 16);
        WIDE_READ(a0, am0, 0);
        WIDE_READ(a1, am1, 0);
        // fragment (k step s, column block c) is piece s rb + c; blocks past the rank read pieces past it, their sums are dropped
        const uint32_t ab1 = ab + rb * 1024;
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            WIDE_READ(b[2 * c], ab, c * 1024);
            WIDE_READ(b[2 * c + 1], ab1, c * 1024);
        }
    };
    // all of them have returned; tied to the registers they fill (also behind the loop, whose last reads nobody uses)
    auto landed = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(xa), "+v"(xb), "+v"(ra), "+v"(rq), "+v"(a0), "+v"(a1));
        asm volatile("" : "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]), "+v"(b[4]), "+v"(b[5]), "+v"(b[6]), "+v"(b[7]), "+v"(b[2 * RB - 8]),
                         "+v"(b[2 * RB - 7]), "+v"(b[2 * RB - 6]), "+v"(b[2 * RB - 5]), "+v"(b[2 * RB - 4]), "+v"(b[2 * RB - 3]), "+v"(b[2 * RB - 2]), "+v"(b[2 * RB - 1]));
    };
    request(gbeg, 0);
    request(gbeg + 1, 1);
    request(gbeg + 2, 2);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * L::kReq) : "memory");
    __builtin_amdgcn_s_barrier();
    read(0);
    int stage = 0;
    for (int g = gbeg; g < gend; ++g) {
        landed();
        const float r[8] = {__uint_as_float(ra.x), __uint_as_float(ra.y), __uint_as_float(ra.z), __uint_as_float(ra.w),
                            __uint_as_float(rq.x), __uint_as_float(rq.y), __uint_as_float(rq.z), __uint_as_float(rq.w)};
        float ta[8], tb[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            ta[2 * i] = bf16lo(xa[i]) * r[2 * i];
            ta[2 * i + 1] = bf16hi(xa[i]) * r[2 * i + 1];
            tb[2 * i] = bf16lo(xb[i]) * r[2 * i];
            tb[2 * i + 1] = bf16hi(xb[i]) * r[2 * i + 1];
        }
#pragma unroll
        for (int c = 0; c < RB; ++c) {
            acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a0), __builtin_bit_cast(bf16x8, b[2 * c]), acc[c], 0, 0, 0);
            acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a1), __builtin_bit_cast(bf16x8, b[2 * c + 1]), acc[c], 0, 0, 0);
        }
        // the next group's operands are asked for here, so that they are on their way from LDS while this group is quantized.  Its stage
        // is complete: behind its requests came the next one's and the code stores of two steps (of fewer at first); and everybody
        // has read this group's, which takes the requests of the group three steps on
        __builtin_amdgcn_sched_barrier(0);
        if (g == gbeg) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L::kReq) : "memory");
        else if (g == gbeg + 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L::kReq + L::kStores) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L::kReq + 2 * L::kStores) : "memory");
        __builtin_amdgcn_s_barrier();
        request(g + 3, stage);
        stage = stage == 2 ? 0 : stage + 1;
        read(stage);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (FMT == 0) {
            // (the words of act_common.h, W4Stage::put)
            uint32_t sa, sb, alo, ahi, blo, bhi;
            const float rcp[2] = {w4_group_rcp(ta, sa), w4_group_rcp(tb, sb)};
            const float(*const runs[2])[8] = {&ta, &tb};
            const act_u32x6 q = w4_codes<2>(runs, rcp);
            w4_run48(q, 0, alo, ahi);
            w4_run48(q, 1, blo, bhi);
            uint32_t wa, wb, wa2, wb2;
            w4.words(alo, ahi, sa, blo, bhi, sb, wa, wb, wa2, wb2);
            WIDE_WRITE(la_out + w4.a, wa);
            WIDE_WRITE(la_out + w4.b, wb);
            WIDE_WRITE(la_out + w4.a2, wa2);
            WIDE_WRITE(la_out + w4.b2, wb2);
            u32x4 v;
            asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(la_out + 16 * lane) : "memory");
            if (lane < kActOutStage / 16) buffer_store_b128<0>(__builtin_bit_cast(buffer_u32x4, v), rs_c, vout, g * (p.Mpad / 32) * kW4ABlock);
        } else {
            uint32_t wa, wb, ba, bb;
            fp4_encode(ta, wa, ba);
            fp4_encode(tb, wb, bb);
            // the four lanes of a block write the same scale byte (an even c8 that of token r8, an odd one that of r8 + 8)
            const int sc = g * p.Mpad * kFp4RowBytes;
            __builtin_amdgcn_raw_buffer_store_b32(wa, rs_c, vca, sc, 0);
            __builtin_amdgcn_raw_buffer_store_b32(wb, rs_c, vcb, sc, 0);
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)((c8 & 1) ? bb : ba), rs_s, vsx, (g >> 2) * p.Mpad * 8 + (g & 3), 0);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    landed();
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // no request is under way when the workgroup's LDS goes to another one
    // housekeeping for the kernel that follows on the stream: its tile arrival counters start at zero
    for (int i = blockIdx.x * 256 + threadIdx.x; i < p.n_zero; i += gridDim.x * 256) p.zero_words[i] = 0u;
    // the run's partial H: fp32 [run][M][rank]
    float *part = p.hpart + (size_t)run * p.M * p.rank;
#pragma unroll
    for (int c = 0; c < RB; ++c)
        if (c < rb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int m = m0 + 4 * blk + v;
                if (m < p.M) part[(size_t)m * p.rank + 16 * c + row] = acc[c][v];
            }
#endif
}

template <int FMT>
hipError_t launch_wide(const ActParams &p, hipStream_t stream) {
    auto k = act_wide_kernel<FMT>;
    constexpr int bytes = WideLds<FMT>::kBytes;
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), bytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)((p.M + kActWideTokens - 1) / kActWideTokens * p.chunks)), dim3(256), bytes, stream, p);
    return hipGetLastError();
}

// H and its bf16 parts from the runs' partial sums [runs][rows][rank], added in run order: four columns of a token per thread, one
// wavefront per workgroup, so that a small launch reaches every CU
__global__ __launch_bounds__(64) void act_sum_h_kernel(const float *hpart, int runs, int M, int rows, int rank, float *H, uint8_t *hfrag) {
    const int quads = rank / 4, idx = blockIdx.x * 64 + threadIdx.x;
    if (idx >= M * quads) return;
    const int m = idx / quads, col = 4 * (idx - m * quads);
    const size_t at = (size_t)m * rank + col, stride = (size_t)rows * rank;
    float4 h = make_float4(0.f, 0.f, 0.f, 0.f);
    constexpr int kBatch = 8;      // runs that are requested before the first addition waits
    for (int c0 = 0; c0 < runs; c0 += kBatch) {
        float4 t[kBatch];
#pragma unroll
        for (int c = 0; c < kBatch; ++c) t[c] = *reinterpret_cast<const float4 *>(hpart + (c0 + c < runs ? c0 + c : c0) * stride + at);
#pragma unroll
        for (int c = 0; c < kBatch; ++c)
            if (c0 + c < runs) { h.x += t[c].x; h.y += t[c].y; h.z += t[c].z; h.w += t[c].w; }
    }
    const uint32_t hi0 = bf16_rne_pair(h.x, h.y), hi1 = bf16_rne_pair(h.z, h.w);
    const uint32_t lo0 = bf16_rne_pair(h.x - bf16lo(hi0), h.y - bf16hi(hi0)), lo1 = bf16_rne_pair(h.z - bf16lo(hi1), h.w - bf16hi(hi1));
    *reinterpret_cast<float4 *>(H + at) = h;
    unsigned char *o = hfrag + 2 * (col & 7);
    *reinterpret_cast<uint2 *>(o + hfrag_offset(rank, m, col, 0)) = make_uint2(hi0, hi1);
    *reinterpret_cast<uint2 *>(o + hfrag_offset(rank, m, col, 1)) = make_uint2(lo0, lo1);
}

}  // namespace

hipError_t launch_act_wide(const ActParams &p, hipStream_t stream) {
    if (p.M <= 0) return hipSuccess;
    if ((p.fmt != 0 && p.fmt != 1) || p.K != p.G * kGroup || p.rank <= 0 || p.rank > 128 || p.rank % 16 || p.Mpad % kRowPad || p.Mpad < p.M || (p.fmt == 1 && !p.sx) || !p.hpart ||
        p.chunks < 1 || p.gchunk < 1 || (size_t)p.gchunk * p.chunks < (size_t)p.G || (p.chunks - 1) * p.gchunk >= p.G || (size_t)p.K * p.Mpad >= ((size_t)1 << 31))
        return hipErrorInvalidValue;
    return p.fmt == 0 ? launch_wide<0>(p, stream) : launch_wide<1>(p, stream);
}

hipError_t launch_act_sum_h(const ActParams &p, int rows, hipStream_t stream) {
    if (p.M <= 0 || p.rank <= 0) return hipSuccess;
    if (!p.hpart || p.chunks < 1 || rows < p.M) return hipErrorInvalidValue;
    hipLaunchKernelGGL(act_sum_h_kernel, dim3((unsigned)(((size_t)p.M * (p.rank / 4) + 63) / 64)), dim3(64), 0, stream, p.hpart, p.chunks, p.M, rows, p.rank, p.H, p.hfrag);
    return hipGetLastError();
}

}  // namespace svdq
