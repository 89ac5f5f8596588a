// W4A4 GEMM for launches between the small tiles of gemm_w4a4_kpar_kernel.hip and the 128 x 256 tiles of gemm_w4a4_kernel.hip: the
// same arithmetic (exact group sums from the block-scaled MFMA, scale tiles from an f16 MFMA, one FMA per partial sum; arXiv
// 2411.05007 Eq. 5), tiles of 128 x 32 C whose width fits the launch to the chip.
//
// A CU runs this loop at full speed with two wavefronts on every SIMD and at half of it with one, so a launch of few tiles
// needs tiles that all CUs get the same number of, and eight wavefronts on each.  The four wavefronts of a share own the
// tile's 4 x C blocks, C each: wavefront (rw, cw) has row blocks 2 rw, 2 rw + 1 of C / 2 columns, and of an odd last column one
// block more.  Two such shares of four wavefronts take the even and the odd groups of K and meet once, in LDS: one workgroup
// per CU.  Operands go from memory straight into a four-stage LDS ring
// with direct-to-LDS loads, three groups ahead, one barrier per group; unlike the K-sharing wavefronts of the small tiles, which
// stream everything from the L2 by themselves, the wavefronts of a share read the same blocks.
// A wavefront's instruction stream is a chain of slots, one per 32 x 32 block, column by column, as in gemm_w4a4_kernel.hip:
//     MFMA A_g(next block) | 16 FMAs of this block | MFMA S_g(next block)
// with the weight block two columns ahead on its way from LDS and the next column's spread to six bits.  Bound: by no unit.  At M =
// 512, K = 3072, N = 9216 (27.0 us) and M = 4096, K = 4608, N = 1152 (32.8 us) the matrix cores are busy 23 and 30 % of the launch and the
// vector ALU 43 and 53 % (the 128 x 256 tiles: 40 and 57 %), the L2 delivers 8 TB/s, and the wavefronts wait for 59 and 53 % of their
// time.  About 7 us are start, low-rank product, meeting and stores; in what is left a SIMD's slot takes about 83 and 72 ns, where a full
// round of the large tiles takes about 55.  One barrier per group spans both shares, so that the two wavefronts of a SIMD enter
// every step together, which is the likely cause, not shown.  No part alone is: copies of the kernel without the requests, the LDS
// reads, the scale tiles or the barrier were at most 10 % faster each, without the spreading none; one row block of C columns to a
// wavefront (twice the spreading), five stages of the ring instead of four, and requests that always hit the L2 change nothing.
// us per forward, where the rule takes it: layout.h, plan_small_int4.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <utility>

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
typedef __attribute__((address_space(3))) void *lds_ptr;

constexpr int kFmtE2M3 = 2;                 // operand format selector of the instruction
constexpr int kScaleBytes = 0x8082;         // block scales 2^3 and 2^1, as in gemm_w4a4_kernel.hip

template <int C>
struct MidTile {
    static constexpr int KS = 2;                                                // shares of K
    static constexpr int kBM = 128, kBN = 32 * C;
    static constexpr int kABytes = 4 * kW4ABlock;                               // 7168
    static constexpr int kPieces = mid_pieces(C);                               // a kilobyte each: activation blocks, then weight blocks
    static constexpr int kReq = (kPieces + 3) / 4;                              // direct-to-LDS requests per wavefront and group
    static constexpr int kStage = kReq * 4096;
    static constexpr int kStages = 4;
    static constexpr int kRing = KS * kStages * kStage;
    static constexpr int kCW = C / 2, kX = C % 2;                               // a wavefront's whole columns (two blocks each), and the odd one (one block)
    static constexpr int kCols = kCW + kX;
    static constexpr int kMeet = 8 * kCols * 4096;                // share 0 finishes the first row block and the odd column, share 1 the second
    static constexpr int kOutWave = 32 * (kCW * 64 + 16);
    static constexpr int kOut = 4 * KS * kOutWave;
    static constexpr int kMax = kMeet > kOut ? kMeet : kOut;
    static constexpr int kLdsBytes = kRing > kMax ? kRing : kMax;
    static_assert((C == 5 || C == 6) && kReq <= C && kLdsBytes <= kLdsBytesPerCU, "");
};

template <typename F, int... t>
__device__ __forceinline__ void mid_each(F &f, std::integer_sequence<int, t...>) { (f(std::integral_constant<int, t>{}), ...); }

// RUNS: H comes as the partial sums of the activation kernel's runs (else ready-made)
template <int C, bool RUNS>
__global__ __launch_bounds__(512, 1) void gemm_w4a4_mid_kernel(GemmW4Params p) {
#ifdef __HIP_DEVICE_COMPILE__      // (the host pass cannot check the asm operands below and would drop the kernel's launch stub without a word)
    using T = MidTile<C>;
    constexpr int KS = T::KS;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w4 = wave & 3, rw = w4 & 1, cw = w4 >> 1, share = wave >> 2;
    auto row_block = [&](int r) { return 2 * rw + (r ^ cw); };      // (the first is the one that the odd column's block belongs to)
    const int li = lane & 31, lh = lane >> 5;
    const int tiles_m = (p.M + T::kBM - 1) / T::kBM, tiles_n = (p.N + T::kBN - 1) / T::kBN;
    int tile_m, tile_n;
    kpar_tile_of((int)blockIdx.x, tiles_m, tiles_n, 4 * kW4ABlock, C * kW4BBlock / 2, tile_m, tile_n);
    const int gm0 = tile_m * T::kBM, gn0 = tile_n * T::kBN;      // rows: inside the padded rows; columns: the last tile may reach past the padded ones

    // ---- memory -> LDS: the tile's four activation blocks and its weight blocks are contiguous in memory, one kilobyte piece after the
    // other dealt to the share's four wavefronts; weight blocks past the padded columns are not asked for (layout.h, mid_piece)
    const __amdgpu_buffer_rsrc_t rs_a = make_rsrc(p.xa, w4_a_bytes(p.G, p.Mpad));
    const __amdgpu_buffer_rsrc_t rs_b = make_rsrc(p.wb, w4_b_bytes(p.G, p.Npad));
    const int a_stride = (p.Mpad / 32) * kW4ABlock, b_stride = (p.Npad / 64) * kW4BBlock;
    int piece_off[T::kReq], piece_stride[T::kReq], piece_lane[T::kReq];
    __amdgpu_buffer_rsrc_t piece_rs[T::kReq];
#pragma unroll
    for (int k = 0; k < T::kReq; ++k) {
        const int j = w4 + 4 * k;
        const bool is_a = j < 7;
        const MidPiece piece = mid_piece(j, lane, T::kPieces, gm0, gn0, p.Npad);
        piece_off[k] = piece.base;
        piece_stride[k] = is_a ? a_stride : b_stride;
        piece_rs[k] = is_a ? rs_a : rs_b;
        piece_lane[k] = piece.lane;      // (or beyond the buffer, which is smaller than 2^31 bytes)
    }
    const int steps = (p.G + KS - 1) / KS, own = (p.G - share + KS - 1) / KS;      // the workgroup's steps, and those in which this share has a group
    unsigned char *ring = lds + share * (T::kStages * T::kStage);
    auto dma_part = [&](int step, int stage, int k) {
        const int g = step * KS + share;
        // past the end: a lane offset beyond the buffer, which asks the memory for nothing (never read)
        const int past = g < p.G ? 0 : (int)0x80000000u;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(piece_rs[k], (lds_ptr)(ring + stage * T::kStage + (w4 + 4 * k) * 1024), 16, piece_lane[k] | past,
                                                 piece_off[k] + (g < p.G ? g : 0) * piece_stride[k], 0, 0);
    };
#pragma unroll
    for (int i = 0; i < T::kStages - 1; ++i)
#pragma unroll
        for (int k = 0; k < T::kReq; ++k) dma_part(i, i, k);
    __builtin_amdgcn_sched_barrier(0);      // the first operands are requested before H and L2

    // ---- bias and low-rank product: the accumulators start as bias + H L2 (share s has rank steps s, s + KS, ...)
    // slot t: row block t % 2 of the wavefront, column t / 2 (the last slot of an odd C: the odd column)
    float acc[C][16];
    auto col_block = [&](int q) { return q < T::kCW ? cw * T::kCW + q : C - 1; };
    {
        typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
        floatx16 lr[C];
        uint32_t col[T::kCols];
#pragma unroll
        for (int q = 0; q < T::kCols; ++q) {
            const int n = gn0 + 32 * col_block(q) + li;
            col[q] = (uint32_t)(n < p.Npad ? n : p.Npad - 1);      // (columns past the padded ones: loaded for nothing, never stored)
            const float b = share == 0 ? p.bias[col[q]] : 0.f;
            lr[2 * q] = floatx16{b, b, b, b, b, b, b, b, b, b, b, b, b, b, b, b};
            if (q < T::kCW) lr[2 * q + (q < T::kCW ? 1 : 0)] = lr[2 * q];
        }
        struct RankStep { uint4 hi[2], lo[2], b[T::kCols]; };
        auto load_rank = [&](RankStep &o, int ks) {
#pragma unroll
            for (int q = 0; q < T::kCols; ++q) o.b[q] = *reinterpret_cast<const uint4 *>(p.l2t + (col[q] * (uint32_t)p.rank + (uint32_t)(ks * 16 + 8 * lh)));
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int m = gm0 + 32 * row_block(r) + li;
                if constexpr (RUNS) {
                    kpar_split_h(kpar_sum_h<4>(p.hpart, p.runs, p.Mpad, p.rank, m, 16 * ks + 8 * lh), o.hi[r], o.lo[r]);
                } else {
                    const unsigned char *h = p.hfrag + hfrag_offset(p.rank, m, 16 * ks + 8 * lh, 0);
                    o.hi[r] = *reinterpret_cast<const uint4 *>(h);
                    o.lo[r] = *reinterpret_cast<const uint4 *>(h + 1024);
                }
            }
        };
        // (a step's operands are requested before the step in front of it is multiplied)
        const int last = p.rank / 16;
        RankStep e, o;
        if (share < last) load_rank(e, share);
        for (int ks = share; ks < last; ks += KS) {
            if (ks + KS < last) load_rank(o, ks + KS);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < C; ++t) {
                lr[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, e.hi[t & 1]), __builtin_bit_cast(bf16x8_t, e.b[t / 2]), lr[t], 0, 0, 0);
                lr[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, e.lo[t & 1]), __builtin_bit_cast(bf16x8_t, e.b[t / 2]), lr[t], 0, 0, 0);
            }
            e = o;
        }
#pragma unroll
        for (int t = 0; t < C; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = lr[t][v];
    }

    // ---- LDS -> registers: reads written as instructions of their own, with explicit waits (the compiler would make every LDS
    // read wait for all outstanding memory-to-LDS requests); a wavefront's LDS operations complete in order
    const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)ring;
    const int h0 = (gn0 / 32) & 1;      // the tile starts in the first or second half of a weight block
    auto half_block = [](int h) { return (uint32_t)((h >> 1) * kW4BBlock + (h & 1) * 1024); };
    auto half_scale = [](int h) { return (uint32_t)((h >> 1) * kW4BBlock + kW4BCodes + (h & 1) * 128); };
    const uint32_t la_a[2] = {base + row_block(0) * kW4ABlock + 24 * lane, base + row_block(1) * kW4ABlock + 24 * lane};
    const uint32_t la_sx[2] = {base + row_block(0) * kW4ABlock + kW4ACodes + 4 * li, base + row_block(1) * kW4ABlock + kW4ACodes + 4 * li};
    // even columns of the wavefront, odd ones, the odd column of the tile
    const int hw = h0 + cw * T::kCW;
    const uint32_t la_b[3] = {base + T::kABytes + half_block(hw) + 16 * lane, base + T::kABytes + half_block(hw + 1) + 16 * lane, base + T::kABytes + half_block(h0 + C - 1) + 16 * lane};
    const uint32_t la_sw[3] = {base + T::kABytes + half_scale(hw) + 4 * li, base + T::kABytes + half_scale(hw + 1) + 4 * li, base + T::kABytes + half_scale(h0 + C - 1) + 4 * li};
    constexpr auto kind = [](int q) { return q < T::kCW ? q & 1 : 2; };              // which of the three a column takes,
    constexpr auto pair = [](int q) { return q < T::kCW ? q / 2 : 0; };              // and how many blocks behind it
    struct AFrag { u32x2 d[3]; };
    struct BFrag { uint32_t d[6]; };
#define MID_READ_A(F, ADDR) \
    asm volatile("ds_read_b64 %0, %3\n\tds_read_b64 %1, %3 offset:8\n\tds_read_b64 %2, %3 offset:16" : "=&v"(F.d[0]), "=&v"(F.d[1]), "=&v"(F.d[2]) : "v"(ADDR))
#define MID_READ_SX(X, ADDR) asm volatile("ds_read2st64_b32 %0, %1 offset0:0 offset1:0" : "=v"(X) : "v"(ADDR))
#define MID_READ_SW(X, ADDR, PAIR) asm volatile("ds_read2st64_b32 %0, %1 offset0:%2 offset1:%2" : "=v"(X) : "v"(ADDR), "n"((PAIR) * (kW4BBlock / 256)))
#define MID_READ_B(Q, ADDR, PAIR) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(Q) : "v"(ADDR), "n"((PAIR) * kW4BBlock))
    auto expand = [&](BFrag &f, const u32x4 &q) {
        f.d[0] = q.x & ~kW4Z0;
        f.d[1] = q.y & ~kW4Z1;
        f.d[2] = (q.x & kW4Z0) | (q.y & kW4Z1);
        f.d[3] = q.z & ~kW4Z0;
        f.d[4] = q.w & ~kW4Z1;
        f.d[5] = (q.z & kW4Z0) | (q.w & kW4Z1);
    };
    auto op_a = [&](const AFrag &f) { return intx8{(int)f.d[0].x, (int)f.d[0].y, (int)f.d[1].x, (int)f.d[1].y, (int)f.d[2].x, (int)f.d[2].y, 0, 0}; };
    auto op_b = [&](const BFrag &f) { return intx8{(int)f.d[0], (int)f.d[1], (int)f.d[2], (int)f.d[3], (int)f.d[4], (int)f.d[5], 0, 0}; };
    auto op_s = [&](u32x2 x) { return __builtin_bit_cast(halfx4, x); };
    const floatx16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    int scales = kScaleBytes;
    asm volatile("" : "+v"(scales));      // one vector register for good (the scale operand cannot be a constant)
#define MID_SB() __builtin_amdgcn_sched_barrier(0)
#define MID_MFMA_A(DST, AF, BF)                                                                                                         \
    DST = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(op_a(AF), op_b(BF), zero16, kFmtE2M3, kFmtE2M3, 0, scales, 1, scales);       \
    asm volatile("" : "+v"(DST), "+v"(sg))
#define MID_MFMA_S(CBLK, SX, SW)                                                        \
    asm volatile("" : "+v"(acc[CBLK][0]), "+v"(acc[CBLK][15]), "+v"(SX));               \
    sg = __builtin_amdgcn_mfma_f32_32x32x8f16(op_s(SX), op_s(SW), zero16, 0, 0, 0);     \
    asm volatile("" : "+v"(sg))

    // LDS reads of a slot, in issue order: a column's first slot asks for the weight block two columns on, its last slot for the
    // scales two columns on, slot kTA for both activation blocks of the next group and their scales (eight reads).  The waits name
    // how many newer reads may still be in flight (at most 15 can be named).
    constexpr int kTA = 1, NC = T::kCols;
    constexpr auto wrap = [](int t) { return (t + 2 * C) % C; };
    constexpr auto col_first = [](int q) { return q >= 0 ? 2 * q : 2 * (q + NC) - C; };                                  // (q < 0: of the step before)
    constexpr auto col_last = [](int q) { return q >= 0 ? (q < T::kCW ? 2 * q + 1 : 2 * q) : (q + NC < T::kCW ? 2 * (q + NC) + 1 : 2 * (q + NC)) - C; };
    constexpr auto is_first = [](int t) { return t % 2 == 0; };
    constexpr auto is_last = [](int t) { return t % 2 == 1 || t == 2 * T::kCW; };
    constexpr auto reads_a = [wrap](int t) { return wrap(t) == kTA ? 8 : 0; };
    constexpr auto reads_in = [wrap, is_first, is_last, reads_a](int t) { return (is_first(wrap(t)) ? 1 : 0) + (is_last(wrap(t)) ? 1 : 0) + reads_a(t); };
    constexpr auto reads_between = [reads_in](int from, int to) {      // slots from .. to, both included
        int n = 0;
        for (int t = from; t <= to; ++t) n += reads_in(t);
        return n;
    };
    constexpr auto at_most_15 = [](int n) { return n < 15 ? n : 15; };

    AFrag af[2][2];
    u32x2 sxr[2][2], swr[2];
    u32x4 braw[2];
    BFrag bfr[2];
    floatx16 ag[2], sg;
    uint32_t st_cur = 0, st_nxt = T::kStage;      // byte offsets of the stages of this step and the next
    int st_free = T::kStages - 1;                 // the stage that this step's requests fill
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    MID_READ_A(af[0][0], la_a[0]);
    MID_READ_A(af[0][1], la_a[1]);
    MID_READ_SX(sxr[0][0], la_sx[0]);
    MID_READ_SX(sxr[0][1], la_sx[1]);
    MID_READ_B(braw[0], la_b[kind(0)], 0);
    MID_READ_SW(swr[0], la_sw[kind(0)], 0);
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(af[0][0].d[0]), "+v"(af[0][0].d[1]), "+v"(af[0][0].d[2]), "+v"(af[0][1].d[0]), "+v"(af[0][1].d[1]), "+v"(af[0][1].d[2]),
                 "+v"(sxr[0][0]), "+v"(sxr[0][1]), "+v"(braw[0]), "+v"(swr[0]));
    expand(bfr[0], braw[0]);
    sg = zero16;
    MID_MFMA_A(ag[0], af[0][0], bfr[0]);
    sg = __builtin_amdgcn_mfma_f32_32x32x8f16(op_s(sxr[0][0]), op_s(swr[0]), zero16, 0, 0, 0);
    asm volatile("" : "+v"(sg));
    MID_READ_B(braw[1], la_b[kind(1)], pair(1));      // as the last column's slots of a step before the first would leave them
    MID_READ_SW(swr[1], la_sw[kind(1)], pair(1));
    MID_SB();

    // P: parity of the step; slots and columns are counted through two steps, so that the double buffers follow their parity
    auto body = [&](int step, auto parity) {
        constexpr int P = decltype(parity)::value;
        auto slot = [&](auto tag) {
            constexpr int t = decltype(tag)::value, cur = (P * C + t) & 1, nxt = cur ^ 1;      // block t's group sums, the next block's
            constexpr int q = t / 2, qc = (P * NC + q) & 1, qn = qc ^ 1;                        // this column's registers, the next column's
            constexpr int t1 = (t + 1) % C, r1 = t1 & 1, PA = t == C - 1 ? P ^ 1 : P;           // the next block, its group
            constexpr bool turn = t1 % 2 == 0;                                                  // it is the first of a column
            MID_SB();
            if constexpr (t == C - 1)
                asm volatile("s_waitcnt lgkmcnt(%8)" : "+v"(af[PA][0].d[0]), "+v"(af[PA][0].d[1]), "+v"(af[PA][0].d[2]), "+v"(af[PA][1].d[0]), "+v"(af[PA][1].d[1]),
                             "+v"(af[PA][1].d[2]), "+v"(sxr[PA][0]), "+v"(sxr[PA][1]) : "n"(at_most_15(reads_between(kTA + 1, C - 2))));
            MID_MFMA_A(ag[nxt], af[PA][r1], bfr[turn ? qn : qc]);
            if constexpr (t == 0) {
                // stage of the next step complete (this wavefront's requests by its wait, the others' by the barrier); the stage of
                // the step before has been read by everybody
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((T::kStages - 3) * T::kReq) : "memory");
                __builtin_amdgcn_s_barrier();
            }
            constexpr int q2 = (q + 2) % NC;      // (of the next step from the last two columns on)
            if constexpr (is_first(t)) MID_READ_B(braw[qc], la_b[kind(q2)] + (q + 2 < NC ? st_cur : st_nxt), pair(q2));
            if constexpr (is_last(t)) MID_READ_SW(swr[qc], la_sw[kind(q2)] + (q + 2 < NC ? st_cur : st_nxt), pair(q2));
            if constexpr (t == kTA) {
                MID_READ_A(af[P ^ 1][0], la_a[0] + st_nxt);
                MID_READ_A(af[P ^ 1][1], la_a[1] + st_nxt);
                MID_READ_SX(sxr[P ^ 1][0], la_sx[0] + st_nxt);
                MID_READ_SX(sxr[P ^ 1][1], la_sx[1] + st_nxt);
            }
            if constexpr (t < T::kReq) dma_part(step + T::kStages - 1, st_free, t);
            // the next column's weight block, asked for in the first slot of the column before this one; in the last slot in front of
            // an odd column also the block of the column behind it, which is multiplied before that column's slot could spread it
            if constexpr (is_first(t) && t != 2 * T::kCW) {
                constexpr int f = col_first(q - 1);
                asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(braw[qn]) : "n"(at_most_15(reads_between(f, t) - 1)));
                expand(bfr[qn], braw[qn]);
            }
            if constexpr (T::kX == 1 && t == C - 2) {
                asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(braw[qc]) : "n"(at_most_15(reads_between(C - 3, t) - 1)));
                expand(bfr[qc], braw[qc]);
            }
            MID_SB();
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = __builtin_fmaf(ag[cur][v], sg[v], acc[t][v]);
            MID_SB();
            if constexpr (turn) {      // its scales, asked for in the last slot of the column before this one
                constexpr int l = col_last(q - 1);
                asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(swr[qn]) : "n"(at_most_15(reads_between(l, t) - 1 - (is_first(wrap(l)) ? 1 : 0))));
            }
            MID_MFMA_S(t, sxr[PA][r1], swr[turn ? qn : qc]);
            MID_SB();
        };
        mid_each(slot, std::make_integer_sequence<int, C>{});
        st_cur = st_nxt;
        st_nxt = st_nxt + T::kStage == T::kStages * T::kStage ? 0u : st_nxt + T::kStage;
        st_free = st_free + 1 == T::kStages ? 0 : st_free + 1;
    };
    // (an odd last step stands behind the loop: a way out between the two would keep two copies of the accumulators)
    for (int i = 0; i + 1 < own; i += 2) {
        body(i, std::integral_constant<int, 0>{});
        body(i + 1, std::integral_constant<int, 1>{});
    }
    if (own & 1) body(own - 1, std::integral_constant<int, 0>{});
    if (own < steps) __builtin_amdgcn_s_barrier();      // an odd number of groups: share 1 has one step less, and every step has a barrier
    // the ring becomes the shares' meeting place: every request of every wavefront must have landed, and every LDS read returned
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" : "+v"(braw[0]), "+v"(braw[1]), "+v"(swr[0]), "+v"(swr[1]) :: "memory");
    __syncthreads();
    int lane_e = lane;      // (the store addresses are worked out here: hoisted above the loop they would be kept across it)
    asm volatile("" : "+v"(lane_e));
    const bool full = gm0 + T::kBM <= p.M && gn0 + T::kBN <= p.N;
    unsigned char *ob = lds + wave * T::kOutWave;
    const float none[1] = {0.f}, nones[T::kCW] = {};
    auto store_row = [&](auto r_tag) {
        constexpr int r = decltype(r_tag)::value;
        gemm_store_wave_tile<1, T::kCW, false>([&](int, int c, int v) { return acc[2 * c + r][v]; }, nones, ob, p.Y, p.M, p.N, gm0 + 32 * row_block(r), gn0 + 32 * cw * T::kCW, full, lane_e);
        if constexpr (r == 0 && T::kX == 1)
            gemm_store_wave_tile<1, 1, false>([&](int, int, int v) { return acc[C - 1][v]; }, none, ob, p.Y, p.M, p.N, gm0 + 32 * row_block(0), gn0 + 32 * (C - 1), full, lane_e);
    };
    using R0 = std::integral_constant<int, 0>;
    using R1 = std::integral_constant<int, 1>;
    // each share leaves the blocks that the other one finishes in LDS in register order
    auto leave = [&](auto r_tag) {
        constexpr int r = decltype(r_tag)::value;
#pragma unroll
        for (int t = r; t < C; t += 2)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                *reinterpret_cast<float4 *>(lds + ((wave * T::kCols + t / 2) * 4 + k) * 1024 + lane_e * 16) = make_float4(acc[t][4 * k], acc[t][4 * k + 1], acc[t][4 * k + 2], acc[t][4 * k + 3]);
    };
    auto take = [&](auto r_tag) {
        constexpr int r = decltype(r_tag)::value;
#pragma unroll
        for (int t = r; t < C; t += 2)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 o = *reinterpret_cast<const float4 *>(lds + (((wave ^ 4) * T::kCols + t / 2) * 4 + k) * 1024 + lane_e * 16);
                acc[t][4 * k] += o.x; acc[t][4 * k + 1] += o.y; acc[t][4 * k + 2] += o.z; acc[t][4 * k + 3] += o.w;
            }
    };
    if (share == 0) leave(R1{});
    else leave(R0{});
    __syncthreads();
    if (share == 0) take(R0{});
    else take(R1{});
    __syncthreads();
    if (share == 0) store_row(R0{});
    else store_row(R1{});
#endif
}

template <int C, bool RUNS>
hipError_t launch_mid(const GemmW4Params &p, hipStream_t stream) {
    using T = MidTile<C>;
    const int tiles_m = (p.M + T::kBM - 1) / T::kBM, tiles_n = (p.N + T::kBN - 1) / T::kBN;
    if (tiles_m * T::kBM > p.Mpad) return hipErrorInvalidValue;      // H is read with plain loads
    if (RUNS && (!p.hpart || p.rank <= 0)) return hipErrorInvalidValue;
    auto k = gemm_w4a4_mid_kernel<C, RUNS>;
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), T::kLdsBytes); e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(tiles_m * tiles_n), dim3(512), T::kLdsBytes, stream, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_w4a4_mid(const GemmW4Params &p, hipStream_t stream) {
    if (p.ksplit != 1 || p.dbg) return hipErrorInvalidValue;
    switch (p.mid_blocks) {
        case 5: return p.runs > 0 ? launch_mid<5, true>(p, stream) : launch_mid<5, false>(p, stream);
        case 6: return p.runs > 0 ? launch_mid<6, true>(p, stream) : launch_mid<6, false>(p, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace svdq
