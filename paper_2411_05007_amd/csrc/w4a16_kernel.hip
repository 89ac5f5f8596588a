// W4A16: the layer with 16-bit activations and the same INT4 weights (arXiv 2411.05007, App. "Implementation
// Details": the inputs of the linear layers in adaptive normalization are kept in 16 bits).
//
//   Y = X^ Q(R) + H L2 + bias,   X^ = bf16(x) * (1 / lambda) in fp32,   Q(R) = s_w[g, n] * codes        (Eq. 5 without Q(X^))
//
// These layers see a handful of rows (one conditioning vector per image), so the kernel streams the weights: the weight
// blocks of the INT4 GEMM are read as they are, once per sixteen rows, and everything else rides along.
//
// Rows go through the matrix core sixteen at a time.  Codes become bf16 (exact: the 16 bytes of one operand lane are
// spread to the 6-bit float form with four AND / AND-OR operations per 16 codes and converted 32 at a time by
// v_cvt_scalef32_pk32_bf16_fp6); X^ is fp32 and goes in as three bf16 parts, each the next eight bits of its significand
// (exact: 24 bits), so that group sums are fp32 sums of exact products, as a vector-ALU kernel's would be.  Up to five
// rows, the three parts of a row are three rows of ONE operand (STACK); more rows take one operand per part.
// Lanes: a lane of a weight block holds 32 codes, channels 32 h .. of column l % 32 (h = l / 32).  v_permlane16_swap
// turns two registers of such lanes (channels 8 j .. and 16 + 8 j .. of all 32 columns, j = 0, 1) into B operands of
// v_mfma_f32_16x16x32_bf16 for columns 0-15 and 16-31 whose k quarter q = l / 16 holds channels 16 q + 8 j .. + 7 of the
// group - the order in which l1s is stored.  X is read to match: a lane takes 16 neighbouring channels of one row, and
// the same registers multiply l1s: H = X l1s of the workgroup's rows comes out of the same loop.
// Work split: a workgroup owns 32 CB columns, wavefront w takes groups w, w + W, ... for all of them, the operands of
// its next group requested while it works on this one; a group's scale is one FMA per output; behind the loop the
// wavefronts' shares of H meet in LDS, H L2 is one or two more steps of the same MFMA, and the wavefronts' sums meet in
// LDS, both in wavefront order (deterministic).
// Up to five rows the parts of X^ (and X itself, for H) are made once per workgroup and lie in LDS, where those of the rows fit it
// and that is the faster side (PARTS; parts_in_lds below): five rows are five of a lane's sixteen operand rows, and a wavefront that makes them in its lanes makes everything three
// times.
// Bound: five rows by the load path (13 requests per group and wavefront: 2.7 us of a CU's time at K = 3072) and 96 vector instructions per
// group (202 with the parts in the loop), more rows by 222 vector and 40 matrix instructions per group, and the fixed parts around the loop.  us
// per forward, rank 32, parts of X^ in the loop -> in LDS: 1 row, K = 3072, N = 18432 11.9 -> 10.8; K = 12288, N = 3072 21.7 -> 16.1; K = N = 8192, rank 16
// 16.4 -> 11.1; K = 4096, N = 1536 9.3 -> 6.6; 5 rows, K = 3072, N = 9216, rank 16 10.3 -> 9.1.  16 rows, K = 3072, N = 18432 14.6.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "buffer.h"
#include "kernels.h"
#include "layout.h"
#include "lds_limit.h"

namespace svdq {
namespace {

typedef uint32_t u32x6 __attribute__((ext_vector_type(6)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));

constexpr int kStackRows = 5;
// LDS of the loop: 1 / lambda of all channels, and behind it the wavefronts' shares of H [wave][16 rows][16 RK + 4]
constexpr int mfma_loop_bytes(int K, int rk, int waves) { return K * 4 + (rk > 0 ? waves * 16 * (16 * rk + 4) * 4 : 0); }
// PARTS: bytes of one part of a row of X^, so that the rows of an operand read fall on distinct banks; and the loop's LDS, [part][row][K] (and, for H, X
// itself behind them) in place of 1 / lambda
constexpr __host__ __device__ int parts_row_bytes(int K) { return 2 * K + 16; }
inline int mfma_parts_bytes(int M, int K, int rk, int waves) {
    const int parts = (rk > 0 ? 4 : 3) * (M < kStackRows ? M : kStackRows) * parts_row_bytes(K), h = rk > 0 ? waves * 16 * (16 * rk + 4) * 4 : 0;
    return parts + h <= kLdsBytesPerCU ? parts + h : parts > h ? parts : h;
}
constexpr int mfma_sums_bytes(int cb, int waves) { return waves * cb * 2 * 16 * 17 * 4; }

// APART: all parts of X^ are made before the first is packed (split8).  PARTS (STACK): they are made once per workgroup, in LDS
template <bool STACK, int CB, int RK, int WAVES, bool APART, bool PARTS>
__global__ __launch_bounds__(WAVES * 64, 1) void w4a16_mfma_kernel(W4A16Params p) {
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];      // 1 / lambda of all channels, later the wavefronts' sums
    constexpr int SETS = STACK ? 1 : 3, RM = STACK ? kStackRows : 16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, q4 = lane >> 4;
    const int n0 = blockIdx.x * CB * 32, m0 = blockIdx.y * RM, G = p.K / 64;
    const int part = STACK ? l16 / kStackRows : 0;      // (operand row 15 carries nothing: part 3, dropped twice, never added)
    const uint32_t drop1 = part >= 1 ? 0xffff0000u : 0u, drop2 = part >= 2 ? 0xffff0000u : 0u;
    const int m_lane = m0 + (STACK ? l16 % kStackRows : l16), row = m_lane < p.M ? m_lane : p.M - 1;      // rows past M repeat the last row; never stored
    // eight fp32 values of a row as the operand registers of the SETS MFMAs; with `careful`, the parts below an infinite value's
    // first are zero (without, they are Inf - Inf)
    auto split8 = [&](const float (&x)[8], u32x4 (&a)[SETS], auto careful) {
        float t[8], u[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            t[e] = x[e] - __uint_as_float(__float_as_uint(x[e]) & (STACK ? drop1 : 0xffff0000u));
            if (decltype(careful)::value && (!STACK || drop1 != 0u) && __builtin_isinf(x[e])) t[e] = 0.f;
            u[e] = t[e] - __uint_as_float(__float_as_uint(t[e]) & (STACK ? drop2 : 0xffff0000u));
        }
        // (Interleaved with the subtractions, the packing waits for the ones right in front of it: K = 3072, N = 18432, rank 32 took 12.8 us
        // instead of 11.9 (1 row), 16.3 instead of 14.6 (16).)
        if constexpr (APART) __builtin_amdgcn_sched_barrier(0);
        auto top = [](float lo, float hi) { return (uint32_t)__builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302); };
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[SETS - 1][e] = top(u[2 * e], u[2 * e + 1]);
            if (!STACK) {
                a[0][e] = top(x[2 * e], x[2 * e + 1]);
                a[SETS / 2][e] = top(t[2 * e], t[2 * e + 1]);
            }
        }
    };
    const __amdgpu_buffer_rsrc_t rs_w = make_rsrc(p.wcodes, w4_b_bytes(G, p.Npad));
    const __amdgpu_buffer_rsrc_t rs_s = make_rsrc(p.sw, (size_t)G * p.Npad * 2);
    const __amdgpu_buffer_rsrc_t rs_x = make_rsrc(p.X, (size_t)p.M * p.K * 2);
    const int vx = (int)(((uint32_t)row * (uint32_t)p.K + 16u * (uint32_t)q4) * 2u);
    // a block past N reads the run's first block: multiplied, never stored
    int first[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) first[cb] = n0 + (n0 + cb * 32 < p.N ? cb * 32 : 0);
    const int rb = p.rank / 16;
    const __amdgpu_buffer_rsrc_t rs_l = make_rsrc(p.l1s, (size_t)p.K * p.rank * 2);
    struct Batch { u32x4 x[2], w[CB], l[RK > 0 ? 2 * RK : 1]; uint16_t s[CB][2]; };
    auto load = [&](int g, auto careful) {      // (careful: for the walk behind the loop)
        Batch t;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            t.w[cb] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_w, 16 * lane, (int)(w4_b_block(g, p.Npad, first[cb]) + 1024 * ((first[cb] % 64) / 32)), 0));
#pragma unroll
            for (int c = 0; c < 2; ++c) t.s[cb][c] = __builtin_amdgcn_raw_buffer_load_b16(rs_s, 2 * l16, (g * p.Npad + first[cb] + 16 * c) * 2, 0);
        }
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (!PARTS || decltype(careful)::value) t.x[j] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_x, vx + 16 * j, g * 128, 0));
#pragma unroll
        for (int i = 0; i < 2 * RK; ++i) {      // blocks past the rank repeat the last one; what they give is dropped
            const int c = i / 2 < rb ? i / 2 : rb - 1;
            t.l[RK > 0 ? i : 0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rs_l, 16 * lane, ((g * 2 + i % 2) * rb + c) * 1024, 0));
        }
        return t;
    };
    Batch cur = load(wave < G ? wave : G - 1, std::false_type{});
    // Everything else that comes from memory is requested right behind: the bias of the outputs this thread will finish,
    // the operands of the wavefront's first low-rank step, 1 / lambda.
    constexpr int kOut = (RM * CB * 32 + WAVES * 64 - 1) / (WAVES * 64);
    float bias[kOut];
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const int n = n0 + (int)(threadIdx.x + i * WAVES * 64) % (CB * 32);
        bias[i] = p.bias[n < p.Npad ? n : 0];
    }
    // low-rank term: 32 columns of H per step, step s by wavefront s % W; the rank is a multiple of 16, its upper end is cut
    // off by zeros
    // (RK > 0: H of the workgroup's rows is made here, behind the loop)
    struct LowRank { float4 h[2]; u32x4 l[CB][2]; };
    const int steps = (p.rank + 31) / 32;
    auto load_lowrank = [&](int s) {
        LowRank t;
        const int j = 32 * s + 8 * q4, jc = j < p.rank ? j : 0;
        if (RK == 0) {
            const float4 *hp = reinterpret_cast<const float4 *>(p.H + (size_t)row * p.rank + jc);
            t.h[0] = hp[0];
            t.h[1] = hp[1];
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int c = 0; c < 2; ++c) t.l[cb][c] = __builtin_bit_cast(u32x4, *reinterpret_cast<const uint4 *>(p.l2t + (size_t)(first[cb] + 16 * c + l16) * p.rank + jc));      // < Npad columns
        return t;
    };
    LowRank low;
    if (wave < steps) low = load_lowrank(wave);
    float *lrinv = reinterpret_cast<float *>(lds);
    // PARTS: eight channels of a row per thread and turn
    const int prow = parts_row_bytes(p.K), have = p.M - m0 < RM ? p.M - m0 : RM;
    if constexpr (PARTS) {
        constexpr int kTurns = 4;      // requested together
        const int chunks = have * (p.K / 8);
        for (int c0 = threadIdx.x; c0 - (int)threadIdx.x < chunks; c0 += kTurns * WAVES * 64) {
            uint4 w[kTurns];
            float4 ra[kTurns], rq[kTurns];
            int at[kTurns];
#pragma unroll
            for (int u = 0; u < kTurns; ++u) {
                if (u > 0 && c0 - (int)threadIdx.x + u * WAVES * 64 >= chunks) break;
                const int c = c0 + u * WAVES * 64 < chunks ? c0 + u * WAVES * 64 : chunks - 1;      // (past the end: the last one again, the same bits)
                const int r = c / (p.K / 8), k = 8 * (c - r * (p.K / 8));
                w[u] = *reinterpret_cast<const uint4 *>(p.X + (size_t)(m0 + r) * p.K + k);
                ra[u] = *reinterpret_cast<const float4 *>(p.rinv + k);
                rq[u] = *reinterpret_cast<const float4 *>(p.rinv + k + 4);
                at[u] = r * prow + 2 * k;
            }
#pragma unroll
            for (int u = 0; u < kTurns; ++u) {
                if (u > 0 && c0 - (int)threadIdx.x + u * WAVES * 64 >= chunks) break;
                const uint32_t xw[4] = {w[u].x, w[u].y, w[u].z, w[u].w};
                const float rr[8] = {ra[u].x, ra[u].y, ra[u].z, ra[u].w, rq[u].x, rq[u].y, rq[u].z, rq[u].w};
                float x[8];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    x[2 * e] = __uint_as_float(xw[e] << 16) * rr[2 * e];
                    x[2 * e + 1] = __uint_as_float(xw[e] & 0xffff0000u) * rr[2 * e + 1];
                }
#pragma unroll
                for (int part = 0; part < 3; ++part) {
                    u32x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        o[e] = (uint32_t)__builtin_amdgcn_perm(__float_as_uint(x[2 * e + 1]), __float_as_uint(x[2 * e]), 0x07060302);
                        x[2 * e] -= __uint_as_float(__float_as_uint(x[2 * e]) & 0xffff0000u);
                        x[2 * e + 1] -= __uint_as_float(__float_as_uint(x[2 * e + 1]) & 0xffff0000u);
                    }
                    *reinterpret_cast<u32x4 *>(lds + part * have * prow + at[u]) = o;
                }
                if (RK > 0) *reinterpret_cast<uint4 *>(lds + 3 * have * prow + at[u]) = w[u];      // X itself, for H
            }
        }
    }
    // (a lane's operand row: part and token; the row that carries nothing and tokens past M read one that is there)
    const int mine = PARTS ? ((part < 3 ? part : 0) * have + (l16 % kStackRows < have ? l16 % kStackRows : have - 1)) * prow + 32 * q4 : 0;
    const int mine_x = PARTS ? (3 * have + (l16 % kStackRows < have ? l16 % kStackRows : have - 1)) * prow + 32 * q4 : 0;
    if constexpr (!PARTS)
        for (int k = 4 * threadIdx.x; k < p.K; k += 4 * WAVES * 64) *reinterpret_cast<float4 *>(lrinv + k) = *reinterpret_cast<const float4 *>(p.rinv + k);
    floatx4 acc[CB][2];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[cb][0] = acc[cb][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto mfma = [](u32x4 a, u32x4 b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0); };
    auto add_lowrank = [&](int s) {
        const bool live = 32 * s + 8 * q4 < p.rank;
        u32x4 a[SETS];
        const float4 ha = low.h[0], hb = low.h[1];
        const float x[8] = {ha.x, ha.y, ha.z, ha.w, hb.x, hb.y, hb.z, hb.w};
        split8(x, a, std::true_type{});
        if (!live)
#pragma unroll
            for (int st = 0; st < SETS; ++st) a[st] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int st = 0; st < SETS; ++st) acc[cb][c] = mfma(a[st], low.l[cb][c], acc[cb][c]);
    };
    __syncthreads();
    if (RK == 0)
        for (int s = wave; s < steps; s += WAVES) {
            if (s >= WAVES) low = load_lowrank(s);
            add_lowrank(s);
        }
    floatx4 hacc[RK > 0 ? RK : 1];
#pragma unroll
    for (int c = 0; c < RK; ++c) hacc[RK > 0 ? c : 0] = floatx4{0.f, 0.f, 0.f, 0.f};
    // one group: X^'s parts, then every column block
    auto multiply = [&](const Batch &t, int g, auto careful) {
        u32x4 a[2][SETS];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (PARTS && !decltype(careful)::value) {
                a[j][0] = *reinterpret_cast<const u32x4 *>(lds + mine + 128 * g + 16 * j);
                continue;
            }
            const float4 *rp = reinterpret_cast<const float4 *>((PARTS ? p.rinv : lrinv) + 64 * g + 16 * q4 + 8 * j);
            const float4 r0 = rp[0], r1 = rp[1];
            const u32x4 w = t.x[j];
            const float x[8] = {__uint_as_float(w.x << 16) * r0.x, __uint_as_float(w.x & 0xffff0000u) * r0.y, __uint_as_float(w.y << 16) * r0.z, __uint_as_float(w.y & 0xffff0000u) * r0.w,
                                __uint_as_float(w.z << 16) * r1.x, __uint_as_float(w.z & 0xffff0000u) * r1.y, __uint_as_float(w.w << 16) * r1.z, __uint_as_float(w.w & 0xffff0000u) * r1.w};
            split8(x, a[j], careful);
        }
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            const u32x4 q = t.w[cb];
            u32x6 d;
            d[0] = q.x & ~kW4Z0;
            d[1] = q.y & ~kW4Z1;
            d[2] = (q.x & kW4Z0) | (q.y & kW4Z1);
            d[3] = q.z & ~kW4Z0;
            d[4] = q.w & ~kW4Z1;
            d[5] = (q.z & kW4Z0) | (q.w & kW4Z1);
            const u32x16 c = __builtin_bit_cast(u32x16, __builtin_amdgcn_cvt_scalef32_pk32_bf16_fp6(d, 8.0f));
            u32x4 op[2][2];      // [k step][columns 0-15, 16-31]
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const auto sw = __builtin_amdgcn_permlane16_swap(c[4 * j + e], c[8 + 4 * j + e], false, false);
                    op[j][0][e] = sw[0];
                    op[j][1][e] = sw[1];
                }
#pragma unroll
            for (int cc = 0; cc < 2; ++cc) {
                const float sc = (float)__builtin_bit_cast(_Float16, t.s[cb][cc]);
                floatx4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int st = 0; st < SETS; ++st) sum = mfma(a[j][st], op[j][cc], sum);
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[cb][cc][v] = __builtin_fmaf(sc, sum[v], acc[cb][cc][v]);
            }
        }
    };
    for (int g = wave; g < G; g += WAVES) {
        const Batch nxt = load(g + WAVES < G ? g + WAVES : g, std::false_type{});      // past the end: this group again, loaded and ignored
#pragma unroll
        for (int j = 0; j < 2; ++j)
            if (PARTS && RK > 0) cur.x[j] = *reinterpret_cast<const u32x4 *>(lds + mine_x + 128 * g + 16 * j);
#pragma unroll
        for (int i = 0; i < 2 * RK; ++i) hacc[RK > 0 ? i / 2 : 0] = mfma(cur.x[i % 2], cur.l[RK > 0 ? i : 0], hacc[RK > 0 ? i / 2 : 0]);
        multiply(cur, g, std::false_type{});
        cur = nxt;
    }
    // An infinite X^ (an infinite input, or one that 1 / lambda carries past fp32) has made NaN of every sum of its row: such a
    // wavefront walks its groups once more, with parts that keep the infinity to the products it belongs to.  A walk of its own,
    // because the test in the loop costs registers (two column blocks, 16 wavefronts: spills) and up to 2 % of a forward; here
    // K = 3072, N = 18432, rank 32 pays, with the low-rank steps' careful parts, 12.68 -> 12.77 us (1 row), 16.08 -> 16.25 (16).
    floatx4 all = acc[0][0] + acc[0][1];
#pragma unroll
    for (int cb = 1; cb < CB; ++cb) all += acc[cb][0] + acc[cb][1];
    const float any = (all[0] + all[1]) + (all[2] + all[3]);
    if (__builtin_expect(__any(any != any), 0)) {
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[cb][0] = acc[cb][1] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (RK == 0)
            for (int s = wave; s < steps; s += WAVES) {
                low = load_lowrank(s);
                add_lowrank(s);
            }
        for (int g = wave; g < G; g += WAVES) multiply(load(g, std::true_type{}), g, std::true_type{});
    }
    // H: the wavefronts' shares meet in LDS behind 1 / lambda; the wavefront of a low-rank step adds up the 32 columns it
    // needs, in wavefront order, as it reads its operand
    constexpr int kHRow = 16 * (RK > 0 ? RK : 1) + 4;
    // (behind 1 / lambda or the parts of X^; in the place of the latter where LDS does not hold both)
    const bool in_place = PARTS && 4 * have * prow + WAVES * 16 * kHRow * 4 > kLdsBytesPerCU;
    if (RK > 0 && in_place) __syncthreads();
    float *hs = PARTS ? reinterpret_cast<float *>(lds + (in_place ? 0 : 4 * have * prow)) : lrinv + p.K;      // [wave][16 rows][kHRow]
#pragma unroll
    for (int c = 0; c < RK; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) hs[(wave * 16 + 4 * q4 + v) * kHRow + 16 * c + l16] = hacc[RK > 0 ? c : 0][v];
    if (RK > 0) {
        __syncthreads();
        if (wave < steps) {      // (RK <= 4: at most two steps)
            const int j = 32 * wave + 8 * q4, jc = j < p.rank ? j : 0;
            float4 ha = make_float4(0.f, 0.f, 0.f, 0.f), hb = ha;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const float4 *hp = reinterpret_cast<const float4 *>(hs + (w * 16 + (STACK ? l16 % kStackRows : l16)) * kHRow + jc);
                const float4 ta = hp[0], tb = hp[1];
                ha.x += ta.x; ha.y += ta.y; ha.z += ta.z; ha.w += ta.w;
                hb.x += tb.x; hb.y += tb.y; hb.z += tb.z; hb.w += tb.w;
            }
            low.h[0] = ha;
            low.h[1] = hb;
            add_lowrank(wave);
        }
    }
    __syncthreads();      // nobody reads 1 / lambda (or the shares of H) any more
    float *sums = reinterpret_cast<float *>(lds);      // [wave][cb][columns 0-15, 16-31][16 rows][17]
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) sums[(((wave * CB + cb) * 2 + c) * 16 + 4 * q4 + v) * 17 + l16] = acc[cb][c][v];
    __syncthreads();
    float y[kOut];
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const int o = threadIdx.x + i * WAVES * 64, cl = o % (CB * 32), m = o / (CB * 32) < RM ? o / (CB * 32) : RM - 1;
        y[i] = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float *s = sums + ((w * CB * 2 + cl / 16) * 16 + m) * 17 + cl % 16;
            y[i] += STACK ? s[0] + (s[kStackRows * 17] + s[2 * kStackRows * 17]) : s[0];
        }
    }
#pragma unroll
    for (int i = 0; i < kOut; ++i) {
        const int o = threadIdx.x + i * WAVES * 64, n = n0 + o % (CB * 32), m = o / (CB * 32);
        if (m < RM && m0 + m < p.M && n < p.N) p.Y[(size_t)(m0 + m) * p.N + n] = __builtin_bit_cast(uint16_t, (__bf16)(y[i] + bias[i]));
    }
}

// Down projection for a handful of rows: H[m][j] = sum_k bf16(x[m][k]) * l1s[k][j] in fp32 (Sec. 4.2: the 16-bit branch,
// lambda^-1 folded into l1s).  The activation kernel gives a whole workgroup to 16 tokens and all columns of H; here a
// workgroup of 16 wavefronts takes 16 rows and 16 columns, wavefront w the groups w, w + 16, ..., three groups' operands
// requested at a time.  l1s is read in its stored fragment order, which with X read to match (lane l: row l % 16,
// channels 16 (l / 16) + 8 s + e of the group for k step s) is the B operand of v_mfma_f32_16x16x32_bf16 as it is; the
// wavefronts' sums are added in wavefront order through LDS.
__global__ __launch_bounds__(1024) void w4a16_proj_kernel(const uint16_t *X, const uint16_t *l1s, float *H, int M, int K, int rank) {
    constexpr int GPW = 3;                                // groups per wavefront whose operands are requested together
    __shared__ float part[16][16][17];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, quarter = lane >> 4;
    const int c = blockIdx.x, m0 = blockIdx.y * 16, G = K / 64, cb = rank / 16;
    const uint16_t *xrow = X + (size_t)(m0 + l16 < M ? m0 + l16 : M - 1) * K + 16 * quarter;      // rows past M repeat the last row; never stored
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int gb = wave; gb < G; gb += 16 * GPW) {
        uint4 f[GPW][2], xv[GPW][2];
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            const int g = gb + 16 * u < G ? gb + 16 * u : G - 1;      // past the end: a valid group, loaded and ignored
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                f[u][s] = *reinterpret_cast<const uint4 *>(l1s + ((((size_t)g * 2 + s) * cb + c) * 64 + lane) * 8);
                xv[u][s] = *reinterpret_cast<const uint4 *>(xrow + g * 64 + 8 * s);
            }
        }
#pragma unroll
        for (int u = 0; u < GPW; ++u) {
            if (gb + 16 * u >= G) break;                                      // uniform over the wavefront
#pragma unroll
            for (int s = 0; s < 2; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, xv[u][s]), __builtin_bit_cast(bf16x8, f[u][s]), acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) part[wave][4 * quarter + v][l16] = acc[v];
    __syncthreads();
    const int o_m = threadIdx.x / 16, o_c = threadIdx.x % 16;
    if (o_m < 16 && m0 + o_m < M) {
        float h = 0.f;
#pragma unroll
        for (int w = 0; w < 16; ++w) h += part[w][o_m][o_c];
        H[(size_t)(m0 + o_m) * rank + 16 * c + o_c] = h;
    }
}

// ---- host side ----------------------------------------------------------------------------------------------------
template <bool STACK, int CB, int RK, int WAVES, bool APART, bool PARTS>
hipError_t launch_mfma_parts(const W4A16Params &p, hipStream_t stream) {
    auto k = w4a16_mfma_kernel<STACK, CB, RK, WAVES, APART, PARTS>;
    static LdsLimit limit;
    if (const hipError_t e = limit.raise(reinterpret_cast<const void *>(k), kLdsBytesPerCU); e != hipSuccess) return e;
    const int rows = STACK ? kStackRows : 16;
    const int loop = PARTS ? mfma_parts_bytes(p.M, p.K, RK, WAVES) : mfma_loop_bytes(p.K, RK, WAVES), sums = mfma_sums_bytes(CB, WAVES), bytes = loop > sums ? loop : sums;
    if (bytes > kLdsBytesPerCU) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, dim3((p.N + 32 * CB - 1) / (32 * CB), (p.M + rows - 1) / rows), dim3(WAVES * 64), bytes, stream, p);
    return hipGetLastError();
}
// Where the parts of X^ lie in LDS (PARTS): where those of the rows fit it, but for
//  - more workgroups than CUs, two of which share a CU without the parts (CB and RK whose registers allow it) and only one with them.  us per forward, parts in the loop |
//    in LDS: 5 rows, K = 2048, N = 36864, rank 32 18.3 | 20.6; 4 rows, K = 2560, N = 24592 14.6 | 15.3; 3 rows, K = 3072, N = 24592 15.9 | 16.7; two on a CU
//    either way: 3 rows, K = 2048, N = 36864 17.3 | 15.1; 2 rows, K = 3072 22.1 | 18.6.  A long K in at most two rounds earns it back up to four rows (K = 4096, N =
//    24592: 2 rows 19.5 | 18.5, 4 rows 20.3 | 20.0; K = 6144 2 rows 26.6 | 24.3), a third round does not (K = 4096, N = 36864: 3 rows 27.8 | 28.2, 4 rows 28.6 | 29.4);
//  - loops of about one group per wavefront, where the turn through LDS and its barrier stand in front of a single step: N = 36864, rank 32, 1 row K = 128 6.8 | 7.4, K = 512
//    7.9 | 8.2, K = 640 8.7 | 8.6; N = 9216, rank 64, 1 row K = 256 4.56 | 4.86; 2 rows, N = 24592, rank 32 K = 320 5.5 | 5.7, K = 512 6.2 | 5.9; 5 rows, N = 24592 K = 128
//    5.6 | 5.4.  Up to 128 columns and rank 32 either does (0 to 2 %).
template <int CB, int RK, int WAVES>
bool parts_in_lds(const W4A16Params &p) {
    const int loop = mfma_parts_bytes(p.M, p.K, RK, WAVES), G = p.K / 64;
    if (loop > kLdsBytesPerCU) return false;
    const bool brief = G <= 8 && (RK > 2 ? p.M * G < 18 : p.M < 4 && p.M * G < 16 && p.N > 128);
    constexpr bool kTwoWithout = WAVES == 8 && (RK == 0 || CB == 1 || (CB == 2 && RK == 2));
    const long wgs = (p.N + 32 * CB - 1) / (32 * CB);
    return !brief && (!kTwoWithout || wgs <= 256 || 2 * loop <= kLdsBytesPerCU || (p.K >= 4096 && p.M <= 4 && wgs <= 512));
}
template <bool STACK, int CB, int RK, int WAVES, bool APART>
hipError_t launch_mfma_apart(const W4A16Params &p, hipStream_t stream) {
    if constexpr (STACK && (WAVES == 8 || (CB == 1 && RK <= 2)))      // (launch_mfma_shape: other launches of sixteen wavefronts are those whose parts do not fit)
        if (parts_in_lds<CB, RK, WAVES>(p)) return launch_mfma_parts<true, CB, RK, WAVES, false, true>(p, stream);
    return launch_mfma_parts<STACK, CB, RK, WAVES, APART, false>(p, stream);
}
// Parts of X^ apart from their packing costs registers.  Sixteen wavefronts have none for it.  Some variants of eight have two
// workgroups on a CU without and one with it, and do it only while one is all there is (M = 54, K = 3840, N = 8960, rank 32, 560
// workgroups: 32.3 us without, 37.9 with; M = 40, K = 3200, N = 12976 29.5 | 33.8).
template <bool STACK, int CB, int RK, int WAVES>
hipError_t launch_mfma(const W4A16Params &p, hipStream_t stream) {
    constexpr bool kTwoFit = (CB == 2 && RK == 2) || (CB == 1 && RK == 4) || (STACK && CB == 3 && RK == 0);
    const long wgs = (long)((p.N + 32 * CB - 1) / (32 * CB)) * ((p.M + (STACK ? kStackRows : 16) - 1) / (STACK ? kStackRows : 16));
    if constexpr (WAVES != 8) return launch_mfma_apart<STACK, CB, RK, WAVES, false>(p, stream);
    if constexpr (kTwoFit)
        if (wgs > 256) return launch_mfma_apart<STACK, CB, RK, WAVES, false>(p, stream);
    return launch_mfma_apart<STACK, CB, RK, WAVES, WAVES == 8>(p, stream);
}
template <bool STACK, int RK>
hipError_t launch_mfma_shape(const W4A16Params &p, hipStream_t stream) {
    // Columns per workgroup: a round of workgroups (one per CU; up to two short ones share a CU, so beyond two rounds parts of
    // rounds count) lasts about 1.2 + CB of what one more 32-column block adds, the 1.2 being X^'s.  (Measured, us, CB = 1,
    // 2, 3, K = 3072, rank 32: 16 rows, N = 18432 21.9, 18.8, 15.9; N = 9216 14.7, 11.8, 15.1; N = 3072 8.8, 10.7, 13.4; 32 rows,
    // N = 18432 34.0, 26.9, 29.5.)
    const int rows = STACK ? kStackRows : 16, passes = (p.M + rows - 1) / rows, blocks = (p.N + 31) / 32;
    int cb = 1;
    double best = 0.0;
    for (int c = 1; c <= 3; ++c) {
        const long wgs = (long)((blocks + c - 1) / c) * passes;
        const double cost = (wgs > 512 && c < 3 ? wgs / 256.0 : (double)((wgs + 255) / 256)) * (1.2 + c);
        if (c == 1 || cost < best) { best = cost; cb = c; }
    }
    // Sixteen wavefronts where a long K meets few columns (K = 12288, N = 3072: 24.6 -> 21.7 us; at K = 3072 eight are as fast),
    // and on two column blocks up to rank 32, whose registers allow it (rank 32, K = N = 12288: 4 rows 30.7 -> 29.1 us, 16 rows
    // 38.5 -> 35.4; K = 6144: 17.8 -> 17.6, 21.8 -> 20.6; rank 64 and three column blocks spill).  Only in one round: two workgroups of
    // eight wavefronts share a CU, where the second one of sixteen waits (eight | sixteen, us: 64 rows, K = N = 8192 46.2 | 51.3; 40 rows,
    // K = 6144, N = 10240 35.0 | 39.6; 4 rows, K = 6144, N = 30720 29.8 | 34.7; 16 rows, K = 12288, N = 30720 66.1 | 72.8)
    // With the parts of X^ in LDS (five rows at most) two column blocks and ranks above 32 are as fast or faster with eight: 3 rows, K = 6144, N = 12288, rank 32
    // 14.1 | 15.3, 1 row, K = N = 12288 20.6 | 21.9, 2 rows, K = 6144, N = 8192, rank 48 13.2 | 17.1; one block up to rank 32 is not: 1 row, K = N = 8192, rank 16 12.2 | 11.1.
    const bool parts = STACK && mfma_parts_bytes(p.M, p.K, RK, 8) <= kLdsBytesPerCU;
    const bool sixteen = p.K >= 6144 && (long)((blocks + cb - 1) / cb) * passes <= 256 && mfma_loop_bytes(p.K, RK, 16) <= kLdsBytesPerCU;
    if (sixteen && cb == 1 && !(parts && RK > 2)) return launch_mfma<STACK, 1, RK, 16>(p, stream);
    if constexpr (RK <= 2)
        if (sixteen && cb == 2 && !parts) return launch_mfma<STACK, 2, RK, 16>(p, stream);
    return cb == 1 ? launch_mfma<STACK, 1, RK, 8>(p, stream) : cb == 2 ? launch_mfma<STACK, 2, RK, 8>(p, stream) : launch_mfma<STACK, 3, RK, 8>(p, stream);
}
template <bool STACK>
hipError_t launch_mfma_rank(const W4A16Params &p, hipStream_t stream) {
    if (p.rank == 0 || !w4a16_makes_h(p.K, p.rank)) return launch_mfma_shape<STACK, 0>(p, stream);
    return p.rank <= 32 ? launch_mfma_shape<STACK, 2>(p, stream) : launch_mfma_shape<STACK, 4>(p, stream);
}

}  // namespace

// Up to rank 64 every workgroup makes H of its rows itself (l1s comes from the L2 beside the weights: K * rank * 2 bytes per
// workgroup), which saves a launch and its wait: one row, N = 18432, rank 32 14.1 -> 12.6 us, rank 64 14.2 -> 13.8;
// sixteen rows 18.2 -> 15.9 and 18.3 (rank 48) -> 16.0.  Wider branches leave H to a launch of its own.
bool w4a16_makes_h(int K, int rank) { return rank <= 64 && mfma_loop_bytes(K, rank <= 32 ? 2 : 4, 8) <= kLdsBytesPerCU; }

hipError_t launch_w4a16_proj(const uint16_t *X, const uint16_t *l1s, float *H, int M, int K, int rank, hipStream_t stream) {
    if (M <= 0 || rank <= 0) return hipSuccess;
    if (K <= 0 || K % 64 || rank % 16) return hipErrorInvalidValue;
    hipLaunchKernelGGL(w4a16_proj_kernel, dim3(rank / 16, (M + 15) / 16), dim3(1024), 0, stream, X, l1s, H, M, K, rank);
    return hipGetLastError();
}

hipError_t launch_w4a16(const W4A16Params &p, hipStream_t stream) {
    if (p.M <= 0) return hipSuccess;
    if (p.K <= 0 || p.K % 64 || p.Npad % kRowPad || p.Npad < p.N || p.rank < 0) return hipErrorInvalidValue;
    if (p.N % 16 || (p.rank > 0 && (!p.l1s || !p.l2t || (!p.H && !w4a16_makes_h(p.K, p.rank))))) return hipErrorInvalidValue;
    return p.M <= kStackRows ? launch_mfma_rank<true>(p, stream) : launch_mfma_rank<false>(p, stream);
}

}  // namespace svdq
