// What the GEMM kernels for launches of few output tiles share: the wavefronts of a workgroup all own the SAME
// (32 RB) x (32 CB) tile and share its K among themselves (wavefront w takes groups w, w + KS, ...), each streaming its
// own operands from the L2 into registers; this is how their partial tiles come together and leave for memory.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "act_common.h"

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
    static constexpr int kWPO = kOctets >= KS ? 1 : KS / kOctets;     // or wavefronts that share an octet
    static constexpr int kCPW = CB / kWPO;                            // column blocks per wavefront
    static constexpr int kOutRow = kCPW * 64 + 16;
    static constexpr int kBytes = kPart + KS * kOPW * 8 * kOutRow;
    static_assert(kOPW * KS == kOctets || kWPO * kOctets == KS, "");
    static_assert(kCPW * kWPO == CB, "");
    static_assert(RB % kPR == 0 && kBytes <= 160 * 1024, "");
};

// acc[r][c][v]: the wavefront's partial tile in the accumulator layout of the 32 x 32 MFMAs (register v of lane l is row
// 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32).  One or two row blocks at a time, every wavefront leaves its partial
// blocks in LDS in register order (16 bytes per lane: no bank conflicts), and each then adds up an equal share of the
// outputs over the wavefronts, in wavefront order, rounds to bf16 (RNE) and stores whole runs of its rows after a turn
// through LDS.
template <int RB, int CB, int KS>
__device__ __forceinline__ void kpar_reduce_store(const float (&acc)[RB][CB][16], unsigned char *lds, uint16_t *Y, int M, int N, int gm0, int gn0,
                                                  int wave, int lane) {
    using T = KparLds<RB, CB, KS>;
    const int li = lane & 31, lh = lane >> 5;
    unsigned char *ob = lds + T::kPart + wave * (T::kOPW * 8 * T::kOutRow);
#pragma unroll
    for (int p0 = 0; p0 < RB; p0 += T::kPR) {
        if (p0 > 0) __syncthreads();      // the partial blocks of the phase before have been read
#pragma unroll
        for (int pr = 0; pr < T::kPR; ++pr)
#pragma unroll
            for (int c = 0; c < CB; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(lds + (((wave * T::kPR + pr) * 4 + q) * CB + c) * 1024 + lane * 16) =
                        make_float4(acc[p0 + pr][c][4 * q], acc[p0 + pr][c][4 * q + 1], acc[p0 + pr][c][4 * q + 2], acc[p0 + pr][c][4 * q + 3]);
        __syncthreads();
        const int c0 = (wave % T::kWPO) * T::kCPW;      // this wavefront's first column block
#pragma unroll
        for (int k = 0; k < T::kOPW; ++k) {
            const int oct = (wave / T::kWPO) * T::kOPW + k;      // rows 8 (oct % 4) .. + 7 of row block oct / 4 of the phase
#pragma unroll
            for (int c = 0; c < T::kCPW; ++c) {
                float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int w = 0; w < KS; ++w) {
                    const float4 t = *reinterpret_cast<const float4 *>(lds + ((w * T::kOctets + oct) * CB + c0 + c) * 1024 + lane * 16);
                    s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
                }
                const uint32_t a = bf16_rne_pair(s.x, s.y), b = bf16_rne_pair(s.z, s.w);
                unsigned char *o = ob + (k * 8 + 4 * lh) * T::kOutRow + (c * 32 + li) * 2;
                *reinterpret_cast<uint16_t *>(o) = (uint16_t)a;
                *reinterpret_cast<uint16_t *>(o + T::kOutRow) = (uint16_t)(a >> 16);
                *reinterpret_cast<uint16_t *>(o + 2 * T::kOutRow) = (uint16_t)b;
                *reinterpret_cast<uint16_t *>(o + 3 * T::kOutRow) = (uint16_t)(b >> 16);
            }
        }
        // only this wavefront touches its block, and the LDS queue of a wavefront is in order: no barrier
        constexpr int kChunks = T::kOPW * 8 * T::kCPW * 4;      // 16-byte chunks; N is a multiple of 16, so a chunk is whole
#pragma unroll
        for (int j = 0; j < (kChunks + 63) / 64; ++j) {
            const int q = lane + 64 * j;
            if (kChunks % 64 && q >= kChunks) break;
            const int row = q / (T::kCPW * 4), ch = q % (T::kCPW * 4);
            const int oct = (wave / T::kWPO) * T::kOPW + row / 8;
            const int grow = gm0 + (p0 + oct / 4) * 32 + 8 * (oct % 4) + row % 8, gcol = gn0 + c0 * 32 + 8 * ch;
            const uint4 v = *reinterpret_cast<const uint4 *>(ob + row * T::kOutRow + ch * 16);
            if (grow < M && gcol < N) *reinterpret_cast<uint4 *>(Y + (size_t)grow * N + gcol) = v;
        }
    }
}

}  // namespace svdq
