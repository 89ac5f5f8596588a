// What the GEMM kernels for launches of few output tiles share: the wavefronts of a workgroup all own the SAME
// (32 RB) x (32 CB) tile and share its K among themselves (wavefront w takes groups w, w + KS, ...), each streaming its
// own operands from the L2 into registers; this is how their partial tiles come together and leave for memory.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "act_common.h"
#include "layout.h"

namespace svdq {

// XCD-aware order of the tiles of a small launch: workgroup b runs on XCD b % 8; every XCD gets a contiguous run of
// tiles (their counts differ by at most one) in an order that walks the shorter operand's side fastest, so that an XCD's
// L2 holds a share of the longer operand and all of the shorter one.  (row_bytes, col_bytes: what one row of the
// activations and one column of the weights cost per group.)
__device__ __forceinline__ void kpar_tile_of(int bid, int tiles_m, int tiles_n, long row_bytes, long col_bytes, int &tile_m, int &tile_n) {
    const int total = tiles_m * tiles_n, q = total / 8, rem = total % 8, x = bid % 8;
    const int id = x * q + (x < rem ? x : rem) + bid / 8;
    if (tiles_m * row_bytes > tiles_n * col_bytes) {
        tile_m = id / tiles_n;
        tile_n = id - tile_m * tiles_n;
    } else {
        tile_n = id / tiles_m;
        tile_m = id - tile_n * tiles_m;
    }
}

template <int RB, int CB, int KS>
struct KparLds {
    static constexpr int kPR = RB >= 2 && CB <= 2 ? 2 : 1;            // row blocks that meet in LDS at a time
    static constexpr int kPart = KS * kPR * CB * 4 * 1024;            // fp32 partial blocks of one phase
    static constexpr int kOctets = kPR * 4;                           // groups of eight rows in a phase
    static constexpr int kOPW = kOctets >= KS ? kOctets / KS : 1;     // octets one wavefront adds up per phase,
    static constexpr int kWPO = kOctets >= KS ? 1 : KS / kOctets < CB ? KS / kOctets : CB;      // or wavefronts that share an octet
    static constexpr int kCPW = CB / kWPO;                            // column blocks per wavefront
    static constexpr int kActive = kOctets / kOPW * kWPO;             // wavefronts that add up a share (all, unless there are more than octets of column blocks)
    static constexpr int kOutRow = kCPW * 64 + 16;
    static constexpr int kBytes = kPart + kActive * kOPW * 8 * kOutRow;
    static_assert(kActive <= KS && kCPW * kWPO == CB, "");
    static_assert(RB % kPR == 0 && kBytes <= 160 * 1024, "");
};

// acc[r][c][v] (32-bit words, fp32 or int32): the wavefront's partial tile in the accumulator layout of the 32 x 32 MFMAs
// (register v of lane l is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32).  One or two row blocks at a time, every
// wavefront leaves its partial blocks in LDS in register order (16 bytes per lane: no bank conflicts), and each then
// adds up an equal share of the outputs over the wavefronts, in wavefront order:
//   take(p0, k, c, s): s = the sums of rows 8 (oct % 4) + 4 (l / 32) .. + 3 of row block p0 + oct / 4, column 32 (c0 + c) + l % 32,
//   where oct, c0 = kpar_share(wave, k);   done(p0): behind the last of a phase.
template <int RB, int CB, int KS>
__device__ __forceinline__ void kpar_share(int wave, int k, int &oct, int &c0) {
    using T = KparLds<RB, CB, KS>;
    oct = (wave / T::kWPO) * T::kOPW + k;
    c0 = (wave % T::kWPO) * T::kCPW;
}
template <typename E> struct alignas(16) Kpar4 { E x, y, z, w; };
template <int RB, int CB, int KS, typename E, typename Take, typename Done>
__device__ __forceinline__ void kpar_meet(const E (&acc)[RB][CB][16], unsigned char *lds, int wave, int lane, Take take, Done done) {
    using T = KparLds<RB, CB, KS>;
    // (a struct, not a vector type: a vector would tie the accumulators to runs of four registers through the whole K loop)
    using e4 = Kpar4<E>;
#pragma unroll
    for (int p0 = 0; p0 < RB; p0 += T::kPR) {
        if (p0 > 0) __syncthreads();      // the partial blocks of the phase before have been read
#pragma unroll
        for (int pr = 0; pr < T::kPR; ++pr)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<e4 *>(lds + (((wave * T::kPR + pr) * 4 + q) * CB + c) * 1024 + lane * 16) =
                        e4{acc[p0 + pr][c][4 * q], acc[p0 + pr][c][4 * q + 1], acc[p0 + pr][c][4 * q + 2], acc[p0 + pr][c][4 * q + 3]};
        __syncthreads();
        if (T::kActive < KS && wave >= T::kActive) continue;
#pragma unroll
        for (int k = 0; k < T::kOPW; ++k) {
            int oct, c0;
            kpar_share<RB, CB, KS>(wave, k, oct, c0);
#pragma unroll
            for (int c = 0; c < T::kCPW; ++c) {
                e4 s{};
#pragma unroll
                for (int w = 0; w < KS; ++w) {
                    const e4 t = *reinterpret_cast<const e4 *>(lds + ((w * T::kOctets + oct) * CB + c0 + c) * 1024 + lane * 16);
                    s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
                }
                take(p0, k, c, s);
            }
        }
        done(p0);
    }
}

// How a wavefront's share of the finished outputs leaves for memory: rounded to bf16 (RNE), whole runs of its rows after
// a turn through its own block of LDS (behind the partial blocks; the LDS queue of a wavefront is in order: no barrier).
template <int RB, int CB, int KS>
struct KparStore {
    using T = KparLds<RB, CB, KS>;
    unsigned char *ob;
    int wave, lane;
    __device__ __forceinline__ KparStore(unsigned char *lds, int wave_, int lane_) : ob(lds + T::kPart + wave_ * (T::kOPW * 8 * T::kOutRow)), wave(wave_), lane(lane_) {}
    __device__ __forceinline__ void put(int k, int c, Kpar4<float> s) {
        const uint32_t a = bf16_rne_pair(s.x, s.y), b = bf16_rne_pair(s.z, s.w);
        unsigned char *o = ob + (k * 8 + 4 * (lane >> 5)) * T::kOutRow + (c * 32 + (lane & 31)) * 2;
        *reinterpret_cast<uint16_t *>(o) = (uint16_t)a;
        *reinterpret_cast<uint16_t *>(o + T::kOutRow) = (uint16_t)(a >> 16);
        *reinterpret_cast<uint16_t *>(o + 2 * T::kOutRow) = (uint16_t)b;
        *reinterpret_cast<uint16_t *>(o + 3 * T::kOutRow) = (uint16_t)(b >> 16);
    }
    __device__ __forceinline__ void store(int p0, uint16_t *Y, int M, int N, int gm0, int gn0) {
        constexpr int kChunks = T::kOPW * 8 * T::kCPW * 4;      // 16-byte chunks; N is a multiple of 16, so a chunk is whole
#pragma unroll
        for (int j = 0; j < (kChunks + 63) / 64; ++j) {
            const int q = lane + 64 * j;
            if (kChunks % 64 && q >= kChunks) break;
            const int row = q / (T::kCPW * 4), ch = q % (T::kCPW * 4);
            int oct, c0;
            kpar_share<RB, CB, KS>(wave, row / 8, oct, c0);
            const int grow = gm0 + (p0 + oct / 4) * 32 + 8 * (oct % 4) + row % 8, gcol = gn0 + c0 * 32 + 8 * ch;
            const uint4 v = *reinterpret_cast<const uint4 *>(ob + row * T::kOutRow + ch * 16);
            if (grow < M && gcol < N) *reinterpret_cast<uint4 *>(Y + (size_t)grow * N + gcol) = v;
        }
    }
};

// fp32 partial tiles whose sum is the output
template <int RB, int CB, int KS>
__device__ __forceinline__ void kpar_reduce_store(const float (&acc)[RB][CB][16], unsigned char *lds, uint16_t *Y, int M, int N, int gm0, int gn0,
                                                  int wave, int lane) {
    KparStore<RB, CB, KS> out(lds, wave, lane);
    kpar_meet<RB, CB, KS>(acc, lds, wave, lane, [&](int, int k, int c, Kpar4<float> s) { out.put(k, c, s); }, [&](int p0) { out.store(p0, Y, M, N, gm0, gn0); });
}

// Columns col .. + 7 of H's row m from the partial H that the runs of the activation kernel left (fp32 [runs][Mpad][rank]), added
// in run order, BATCH runs requested before the first addition waits.
struct KparH { float h[8]; };
template <int BATCH = 4>
__device__ __forceinline__ KparH kpar_sum_h(const float *hpart, int runs, int Mpad, int rank, int m, int col) {
    const size_t at = (size_t)m * rank + col, stride = (size_t)Mpad * rank;
    KparH o{};
    for (int c0 = 0; c0 < runs; c0 += BATCH) {
        float4 t[BATCH][2];
#pragma unroll
        for (int c = 0; c < BATCH; ++c) {
            const float4 *q = reinterpret_cast<const float4 *>(hpart + (c0 + c < runs ? c0 + c : c0) * stride + at);
            t[c][0] = q[0];
            t[c][1] = q[1];
        }
#pragma unroll
        for (int c = 0; c < BATCH; ++c)
            if (c0 + c < runs) {
                o.h[0] += t[c][0].x; o.h[1] += t[c][0].y; o.h[2] += t[c][0].z; o.h[3] += t[c][0].w;
                o.h[4] += t[c][1].x; o.h[5] += t[c][1].y; o.h[6] += t[c][1].z; o.h[7] += t[c][1].w;
            }
    }
    return o;
}
// such values as the bf16 hi and lo parts that the matrix core is fed
__device__ __forceinline__ void kpar_split_h(const KparH &v, uint4 &vhi, uint4 &vlo) {
    uint32_t hi[4], lo[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        hi[e] = bf16_rne_pair(v.h[2 * e], v.h[2 * e + 1]);
        lo[e] = bf16_rne_pair(v.h[2 * e] - bf16lo(hi[e]), v.h[2 * e + 1] - bf16hi(hi[e]));
    }
    vhi = make_uint4(hi[0], hi[1], hi[2], hi[3]);
    vlo = make_uint4(lo[0], lo[1], lo[2], lo[3]);
}
// H of the tile's rows below M (the others' places are left as they are: they only meet outputs that are not stored), left in LDS in
// the operand order of hfrag (rows counted from the tile's first).  All threads take part; ends with a barrier.
// (H is not written to memory here: a store in front of the K loop holds up every later load of its wavefront until memory has
// acknowledged it, 2.5 us per store and wait in the workgroups that wrote it, and so in the launch.)
template <int RB, int KS>
__device__ __forceinline__ void kpar_sum_h_tile(unsigned char *lds, const float *hpart, int runs, int M, int Mpad, int rank, int gm0, int tid) {
    const int octets = rank / 8, rows = M - gm0 < 32 * RB ? M - gm0 : 32 * RB;
    for (int idx = tid; idx < rows * octets; idx += KS * 64) {
        const int m = idx / octets, col = 8 * (idx - m * octets);
        KparH h;      // (a batch beyond the runs asks for the first of them again)
        if (runs <= 2) h = kpar_sum_h<2>(hpart, runs, Mpad, rank, gm0 + m, col);
        else if (KS != 8 || runs <= 4) h = kpar_sum_h<4>(hpart, runs, Mpad, rank, gm0 + m, col);
        else h = kpar_sum_h<8>(hpart, runs, Mpad, rank, gm0 + m, col);
        uint4 hi, lo;
        kpar_split_h(h, hi, lo);
        *reinterpret_cast<uint4 *>(lds + hfrag_offset(rank, m, col, 0)) = hi;
        *reinterpret_cast<uint4 *>(lds + hfrag_offset(rank, m, col, 1)) = lo;
    }
    __syncthreads();
}
// LDS that the sums need
template <int RB> constexpr int kpar_h_bytes(int rank) { return 32 * RB * rank * 4; }

}  // namespace svdq
