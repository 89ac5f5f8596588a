// Native buffer layouts shared by the host packer and the HIP kernels.
//
// Both 4-bit operands are stored "group-major": for every group g of 64 input channels, the blocks of all rows (tokens
// of the activation, output channels of the weight) of that group are contiguous, so the GEMM's K loop streams one
// contiguous slab per operand per step.  The INT4 blocks (activation blocks of 32 rows, weight blocks of 64 columns,
// each with its codes in the matrix instruction's operand order and its fp16 scales) are described further down,
// next to the MXFP4 and 8-bit forms.
//     weight scales wscales[g][n]  (fp16): a plain copy beside the blocks, read by the W4A16 kernels
//     low-rank activations (workspace) H[m][rank] fp32, and the same values split into bf16 hi + lo parts
//         (hi = bf16(h), lo = bf16(h - hi)) in the A-operand order of v_mfma_f32_32x32x16_bf16:
//         hfrag[m / 32][rank step of 16][part][lane = 32 ((j % 16) / 8) + m % 32][8 bf16], so the GEMM loads
//         a ready-made operand with one 16-byte load per lane (hfrag_offset)
//
// Rows are padded to a multiple of 256 so a full tile can always be read; padding rows of the
// weight hold zero codes and zero scales.
//
// The two bf16 low-rank factors are stored in the order the MFMA instructions consume them:
//   l1s  [G][2 (k step)][rank/16 (column block)][64 (lane)][8]  - B operand of
//        v_mfma_f32_16x16x32_bf16 in the activation kernel: lane l, element e of k step s holds
//        L1s[64 g + 16 (l / 16) + 8 s + e][16 c + l % 16]
//   l2   [Npad][rank]  (L2 transposed) - B operand of v_mfma_f32_32x32x16_bf16 in the GEMM (up projection).
#pragma once
#include <stddef.h>
#include <stdint.h>

#ifndef __HIPCC__
#ifndef __host__
#define __host__
#endif
#ifndef __device__
#define __device__
#endif
#endif

namespace svdq {

constexpr int kGroup = 64;
constexpr int kRowPad = 256;        // rows of every group-major tensor are padded to this
constexpr int kMaxRank = 256;

// Byte offset of the 16-byte chunk of hfrag that holds columns 8 (j / 8) .. + 7 of row m; part 0 = hi, 1 = lo.
inline __host__ __device__ size_t hfrag_offset(int rank, int m, int j, int part) {
    const int ks = j / 16, kq = (j % 16) / 8;
    return ((((size_t)(m / 32) * (rank / 16) + ks) * 2 + part) * 64 + (kq * 32 + m % 32)) * 16;
}

inline __host__ __device__ int round_up(int v, int m) { return (v + m - 1) / m * m; }
inline __host__ __device__ size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

inline __host__ __device__ size_t l1s_index(int K, int rank, int k, int j) {
    (void)K;
    const int g = k / 64, kk = k % 64;
    const int blk = kk / 16, s = (kk % 16) / 8, e = kk % 8;
    const int c = j / 16, lane = blk * 16 + (j % 16);
    return ((((size_t)g * 2 + s) * (rank / 16) + c) * 64 + lane) * 8 + e;
}

// ---- INT4 operands of the block-scaled matrix instruction (W4A4 GEMM) ------------------------------------------
// v_mfma_scale_f32_32x32x64_f8f6f4 multiplies one group of 64 channels per instruction.  Its 6-bit float format
// E2M3 (sign, two exponent bits, three mantissa bits) holds every INT4 code exactly: with the exponent bits zero
// the element is sign * mantissa / 8, so code q becomes the six bits  s 0 0 m m m  with m = |q|; the instruction's
// power-of-two block scales (2^3 for each operand) take the two factors 1/8 out again and the fp32 result is the
// exact integer group sum.  Lane l of an operand feeds row (column) l % 32 with the 32 channels of half l / 32 of
// the group, channel e of the half in bits 6 e .. 6 e + 5 of the lane's six registers.
//
//   activation blocks (workspace)  xa[g][m / 32][1792 bytes]: bytes 24 l .. 24 l + 23 = lane l's six registers,
//       bytes 1536 + 4 (m % 32) = the row's fp16 group scale in the low half of a dword whose high half is zero;
//       the last 128 bytes are padding that is never read (a block is seven times 256 bytes so that one LDS
//       address register reaches the scales of every block).  The activation kernel writes this form directly.
//   weight blocks (prepared layer) wb[g][n / 64][2304 bytes], one block per 64 columns (what one wavefront of the
//       GEMM multiplies): bytes 1024 (n % 64 / 32) + 16 l .. + 15 = lane l's 32 codes at FOUR bits each, bytes
//       2048 + 4 (n % 64) = the column's fp16 group scale, again as the low half of a dword.  A scale dword read into
//       both registers of an f16 MFMA operand makes that operand without a vector instruction.
//       The 4 stored bits of a code sit where
//       three AND / AND-OR operations per register pair spread them into the 6-bit form (w4_b_bitpos): of every 16
//       codes = 96 operand bits = registers T0 T1 T2, the stored pair S0 S1 holds T0's and T1's used bits in
//       place, and T2's used bits in the positions that T0 and T1 leave zero (their exponent bits):
//           T0 = S0 & ~Z0,  T1 = S1 & ~Z1,  T2 = (S0 & Z0) | (S1 & Z1).
// A block carries its scales so that one contiguous copy brings everything a 32-row block needs for one group.
constexpr int kW4ACodes = 1536, kW4AUsed = 1664, kW4ABlock = 1792;     // bytes of codes / of codes + scales / of the whole activation block
constexpr int kW4BCodes = 2048, kW4BBlock = 2304;     // bytes of codes / of the whole weight block (64 columns)
constexpr uint32_t kW4Z0 = 0x18618618u;               // exponent-bit positions inside T0 (bits 3, 4 of every 6)
constexpr uint32_t kW4Z1 = 0x86186186u;               // the same inside T1 (T1 starts at bit 32 = bit 2 of element 5)
inline __host__ __device__ size_t w4_a_block(int g, int Mpad, int m) { return ((size_t)g * (Mpad / 32) + m / 32) * kW4ABlock; }
inline __host__ __device__ size_t w4_b_block(int g, int Npad, int n) { return ((size_t)g * (Npad / 64) + n / 64) * kW4BBlock; }
inline __host__ __device__ size_t w4_a_bytes(int G, int Mpad) { return (size_t)G * (Mpad / 32) * kW4ABlock; }
inline __host__ __device__ size_t w4_b_bytes(int G, int Npad) { return (size_t)G * (Npad / 64) * kW4BBlock; }
// Bit position (0..127, inside lane l's 16 bytes of a weight block) of bit b of channel e (0..31) of the lane's half
// group: b = 0..2 are the magnitude bits, b = 3 the sign.
inline __host__ __device__ int w4_b_bitpos(int e, int b) {
    const int pair = e / 16, p = 6 * (e % 16) + (b < 3 ? b : 5);      // position in the 96 operand bits T0 T1 T2
    if (p < 32) return pair * 64 + p;
    if (p < 64) return pair * 64 + p;                                  // S1 bit p - 32
    const int q = p - 64;
    return pair * 64 + (((kW4Z0 >> q) & 1u) ? q : 32 + q);
}
// The 6-bit operand form of code q in [-7, 7] (-8 is not a code of the symmetric quantizer).
inline __host__ __device__ uint32_t w4_e2m3(int q) { return q < 0 ? (32u | (uint32_t)(-q)) : (uint32_t)q; }

// ---- 8-bit setting (one int8 per code, one fp16 scale per token and per output channel) ---------------------
// Both operands in the operand order of v_mfma_i32_32x32x32_i8, whose lane l feeds row (or column) l % 32 with
// the 16 channels 16 (l / 32) .. + 15 of a 32-channel step:
//     codes  c8[k / 32][row / 32][lane = 32 ((k % 32) / 16) + row % 32][16 bytes], byte k % 16
// so one 32-row block of one 32-channel step is one contiguous kilobyte.  Scales: fp16 [rows_pad].
inline __host__ __device__ size_t i8_code_offset(int k, int rows_pad, int row) {
    return ((((size_t)(k / 32) * (rows_pad / 32) + row / 32) * 64 + ((k % 32) / 16) * 32 + row % 32) * 16) + k % 16;
}
// ---- MXFP4 variant (E2M1 elements, blocks of 32 along K, one power-of-two scale byte per block) ----------
// Both operands use the A / B operand order of v_mfma_scale_f32_32x32x64_f8f6f4, whose lane l feeds row (or
// column) l % 32 with the 32 elements of block l / 32 of a 64-channel step:
//     codes   c4[g][row / 32][kb][row % 32][16 bytes], nibble t of the 16 bytes = element k = 64 g + 32 kb + t
//     scales  s4[g / 4][row / 32][kb * 32 + row % 32][g % 4]: one dword per lane carries the scale bytes of
//             four consecutive steps, picked by the instruction's byte selector
// so one 32-row block of one step is one contiguous kilobyte of codes, loaded with one 16-byte load per lane.
constexpr int kFp4Block = 32;
// Loads of the GEMMs that ask for nothing (a step past the wavefront's last, a place of the ring that a tile
// has no block for) get their zeros from a lane offset of 2^31, beyond every buffer.  Their uniform offset stays inside the
// buffer all the same: what a range check makes of one beyond it depends on whether it is part of the check.
//   the step a wavefront's i-th load belongs to (wavefront w of KS has steps w, w + KS, ..., n of them):
inline __host__ __device__ int kpar_step(int wave, int KS, int i, int n) { return i < n ? wave + KS * i : 0; }
//   byte offset of ring place j in a step of its operand (activation blocks, weight blocks, none), for a tile at (gm0, gn0):
inline __host__ __device__ int ring_offset(int j, int frags_a, int frags_b, int gm0, int gn0) {
    return j < frags_a ? gm0 * 32 + j * 1024 : j < frags_a + frags_b ? gn0 * 32 + (j - frags_a) * 1024 : 0;
}
// XCD-aware tile order.  Workgroups are dealt round-robin to the chip's 8 XCDs, each with an L2 of its own; they are
// renumbered so that an XCD owns a contiguous run of tiles (their counts differ by at most one), walked in bands of eight tile
// rows, column by column inside a band: the 64 tiles an XCD runs at a time (two workgroups per CU) are then 8 x 8, the shape with
// the fewest distinct operand blocks (measured on the INT4 GEMM at 1728 tiles: bands of 4, 6, 8, 12 rows miss the L2 for 260,
// 224, 217, 239 MB per launch; bands of 2 to 18 rows run within 1 % of each other).
// Counts that 8 does not divide are renumbered from `from` tiles on.  us per forward in launch order -> renumbered: MXFP4, M = 1663, K = 7936, N = 8480
// (476 tiles) 87.7 -> 74.5, M = 4162, K = 3392, N = 9296 (1221) 111 -> 96.3; INT8, M = 2943, K = 2560, N = 10576 112.9 -> 91.5, M = 1677,
// K = 5888, N = 11328 155 -> 128 (33 launches of both: median 5 % faster, none slower).  The INT4 kernel, bound by power and not by the L2, gains 0 to 6 % above
// 600 tiles (M = 4429, K = 1856, N = 10720 127.6 -> 120; M = 4169, K = 2496, N = 9472 125.6 -> 121.8) and loses 0 to 5 % below (M = 2213, K = 1536,
// N = 6672, 486 tiles 38.4 -> 40.1).
// MXFP4 and INT8 launches below 600 tiles with short rows and up to 4096 columns stay in launch order too, in which the eight rows of a band fall on the eight XCDs, each of which then
// reads its own: 1.7 % faster in the geometric mean of 162 launches (MXFP4, K up to 1536, M = 3270, K = 1536, N = 1872 15.0 in launch order, 15.5 renumbered; INT8, K up to 1024, M = 1823, K = 384,
// N = 2272 13.5 | 14.0).  Longer rows gain by the numbering at every width (K = 2560, 1 to 2.5 %), and so do wider launches (more than 5000 columns 0 to 7 %: INT8, M = 1703, K = 384, N = 8304 21.6 | 20.3).
// `bid`: position in the launch order, 0 <= bid < total = tiles_m * tiles_n.
constexpr int kXcdOrderInt4 = 600;
inline __host__ __device__ int xcd_order_from(bool i8, int G, int N) { return N <= 4096 && G <= (i8 ? 16 : 24) ? 600 : 0; }
inline __host__ __device__ void gemm_tile_of(int bid, int tiles_m, int tiles_n, int from, int &tile_m, int &tile_n) {
    constexpr int kBand = 8;
    const int total = tiles_m * tiles_n, per = total / 8, more = total % 8, xcd = bid % 8;      // the first `more` XCDs own a tile more than the others
    const int id = more == 0 || total >= from ? xcd * per + (xcd < more ? xcd : more) + bid / 8 : bid;
    const int band = id / (kBand * tiles_n);
    const int band_rows = (tiles_m - band * kBand) < kBand ? (tiles_m - band * kBand) : kBand;
    const int in = id - band * kBand * tiles_n;
    tile_m = band * kBand + in % band_rows;
    tile_n = in / band_rows;
}
constexpr int kGemmPlaces = 512;     // places for workgroups of the 128 x 256 tiles: two per CU
constexpr int kFp4RowBytes = 32;     // packed bytes of one row of one 64-channel step
constexpr int kMaxKSplitFp4 = 8;
inline __host__ __device__ size_t fp4_code_offset(int g, int rows_pad, int row, int kb) {
    return ((((size_t)g * (rows_pad / 32) + row / 32) * 2 + kb) * 32 + row % 32) * 16;
}
inline __host__ __device__ size_t fp4_scale_offset(int g, int rows_pad, int row, int kb) {
    return ((((size_t)(g / 4) * (rows_pad / 32) + row / 32) * 64 + kb * 32 + row % 32) * 4) + g % 4;
}
inline __host__ __device__ size_t fp4_scale_bytes(int G, int rows_pad) { return (size_t)((G + 3) / 4) * rows_pad * 8; }

// Launch plan of the MXFP4 GEMM.  A launch with fewer workgroups than the chip has
// places for (two per CU) splits a long K loop over up to four workgroups per tile, each a multiple of four steps
// and at least 32 steps long (measured: at 48 steps per tile the parked partial tiles cost what the shorter loop
// saves; at 192 steps four splits halve the time, eight are slower again); the partial tiles meet in the
// workspace as in the INT4 kernel.  Left to themselves such launches run the kernel whose wavefronts share K
// (plan_kpar_blocks) and split nothing; the workspace keeps room for the split, which a caller can ask for.
struct GemmPlanFp4 {
    int tile;        // 0: 128 x 256, 1: 192 x 192, 2: 192 x 128, 3: 128 x 128
    int tiles, ksplit;
};
inline GemmPlanFp4 plan_gemm_fp4(int M, int N, int G, int ksplit_override = 0, int min_steps = 32, bool i8 = false) {
    GemmPlanFp4 pl;
    pl.tiles = ((M + 127) / 128) * ((N + 255) / 256);
    int s = 1;
    if (pl.tiles <= 128) {                          // measured: with 160 tiles and 72 steps two splits are slower than none
        s = 512 / pl.tiles;
        if (s > 4) s = 4;
        while (s > 1 && G / s < min_steps) --s;
    }
    if (ksplit_override > 0) s = ksplit_override < kMaxKSplitFp4 ? ksplit_override : kMaxKSplitFp4;
    // normalise: splits are multiples of four steps, none empty
    while (s > 1 && (size_t)(s - 1) * (((G + s - 1) / s + 3) / 4 * 4) >= (size_t)G) --s;
    pl.ksplit = s < 1 ? 1 : s;
    pl.tile = 0;
    // The tile shape.  What a launch takes follows the CU with the most tiles, but not all the way (a CU that is done early leaves its share of
    // the L2 to the others): the mean of the tiles per CU and of that number rounded up, times the MFMAs per step of a tile, weighted with
    // what the tile loads per MFMA, and more where no CU has a second tile to fill the first one's waits (192 x 192 tiles, which ask for a
    // step's operands between its products, need that least, and cost more around a short K loop: INT8, M = 1585, K = 1152, N = 4224 20.9 | 19.8 on 128 x 128,
    // MXFP4, M = 4111, K = 1728, N = 6896 50.9 | 49.3 on 128 x 256; more so where they are at most one per CU: INT8, M = 527, K = 640, N = 11136 17.6 | 15.8 on 128 x 128, M = 2080, K = 1664,
    // N = 2976 23.7 | 22.2; less so where a CU has more than four of them and the K loop is longer than their start: INT8, M = 4493, K = 1152, N = 19904 136.8 on 128 x 256 | 124.3, MXFP4, M = 2571, K = 1024, N = 25232
    // 65.9 | 61.2, but M = 4012, K = 384, N = 19552 56.7 | 62.4).  Large INT8 launches of up to seven groups are stores of 16-bit results before all else, which small tiles
    // spread better (M = 3728, K = 64, N = 34544 81.6 on 192 x 192 | 73.3 on 128 x 128).  192-row and 192-column tiles have to fit the padded rows and columns.  Fitted to 1400 launches, G = 1 to 192,
    // of two to four shapes each; up to two 128 x 256 tiles per CU they keep the launches that the others win by less than 3 %.
    // us per forward, 128 x 256 | 192 x 192 | 192 x 128 | 128 x 128, the rule's choice in brackets; MXFP4 rank 32, INT8 rank 16:
    //   M = 4608, K = 3072, N = 9216 (1296 | 1152 | 1728 | 2592 tiles)   97.8 [87.3] 95.7  98.6     157.1 [138.2] 147.5 153.9
    //   M = 3000, K = 3072, N = 9216 (864 | 768 | 1152 | 1728)           65.7 [57.8] 68.3  65.7     101.9 [89.2] 101.9  98.8
    //   M = 1800, K = 3072, N = 12288 (720 | 640 | 960 | 1440)           53.9 [50.9] 55.9  54.9      80.8 [78.5]  81.7  82.5
    //   M = 4608, K = N = 3072 (432 | 384 | 576 | 864)                  [43.8] 43.1  48.8  46.0     [65.6] 64.2   75.6  68.9
    //   M = 4178, K = 3520, N = 5744 (759 | 660 | 990 | 1485)            66.3 [63.5] 68.8  68.2
    //   M = 4406, K = 7168, N = 2304 (315 | 276 | 414 | 630)             75.7  77.2 [70.8] 72.6
    //   M = 907, K = 5952, N = 7216 (232 | 190 | 285 | 456)                                          58.1 [52.5]  61.9  55.8
    //   M = 892, K = 3456, N = 7232 (203 | 190 | 285 | 399)              27.2 [26.0] 30.7  26.4
    //   M = 2048, K = N = 3072 (192 | - | - | 384)                       31.8   -     -   [29.0]     44.4   -      -   [41.5]
    // (the last with the activation kernel of 16-token workgroups)
    if (pl.ksplit == 1) {
        auto cost = [](long tiles, double per_tile, double lone) { return (tiles / 256.0 + (double)((tiles + 255) / 256)) * per_tile * (tiles <= 256 ? lone : 1.0); };
        const int pm = round_up(M, kRowPad), pn = round_up(N, kRowPad), tm = (M + 127) / 128, tm192 = (M + 191) / 192, tn = (N + 127) / 128, tn192 = (N + 191) / 192;
        const int tiles[4] = {pl.tiles, tm192 * 192 <= pm && tn192 * 192 <= pn ? tm192 * tn192 : 0, tm192 * 192 <= pm ? tm192 * tn : 0, tm * tn};
        const double per_tile[4] = {8.0, 9 * (0.89 + (G >= 12 && tiles[1] > 1024 ? 1.2 : 2.0) / (G > 18 ? G : 18)), 6 * 1.05, 4 * (i8 && G < 8 && tiles[3] > 1280 ? 0.95 : 1.07)};
        const double lone192 = G < 67 ? 1.0 + 2.0 / (G > 12 ? G : 12) : 1.03;
        double best = (pl.tiles <= 512 ? 0.97 : 1.0) * cost(pl.tiles, per_tile[0], 1.2);
        for (int t = 1; t < 4; ++t) {
            const double c = cost(tiles[t], per_tile[t], t == 1 ? lone192 : 1.1);
            if (tiles[t] > 0 && c < best) {
                best = c;
                pl.tile = t;
                pl.tiles = tiles[t];
            }
        }
    }
    return pl;
}

// how the activation kernel's launch is cut up (plan_act below)
struct ActPlan {
    int chunks;      // runs per 16-token slice, 1..64
    int gchunk;      // groups per run (the last run may be shorter)
    int waves;       // wavefronts per workgroup: 4 or 8
    // the first `whole` slices of a launch can be cut differently from the rest (or not at all): chunks0 runs of gchunk0 groups
    int whole, chunks0, gchunk0;
    bool deposit;    // the runs' partial H are left for the GEMM to add (plan_act_small)
};
struct WorkspaceFp4 {
    size_t codes_off, bx_off, h_off, hfrag_off, counters_off, partial_off, hpart_off, aflags_off, total;
    int Mpad;
    int n_counters;
    ActPlan act;      // the activation kernel's cut of K
};


// Variants of the GEMM for launches of few tiles: (32 RB) x 64 tiles, KS wavefronts per workgroup that share K; kKparNarrow: 32 x 32 tiles,
// sixteen wavefronts.
enum KparVariant { kKparNone = 0, kKpar1x8, kKpar2x8, kKpar2x4, kKpar4x8, kKpar4x4, kKparNarrow, kKparVariants };
// INT4.  Small tiles where the launch is short of workgroups, larger ones where it is not (fewer bytes from the L2 per
// product); eight wavefronts while one such workgroup per CU is all there is, four (two workgroups per CU) beyond.
// Measured, us per forward at rank 32 with the kernel of 128 x 256 tiles (K loops split over workgroups) first:
//   M = 256, K = N = 1152 (72 tiles of 64 x 64): 27.8; 1x8 11.6, 2x8 12.5, 2x4 13.3.   M = 64, K = 12288, N = 3072 (48): 49.9; 1x8 20.7, 2x8 24.5
//   M = 300, K = 3072, N = 2064 (165): 35.6; 1x8 17.5, 2x8 15.6, 2x4 17.1.              M = 128, K = 3072, N = 9216 (288): 31.5; 2x8 19.1, 2x4 17.3
//   M = 512, K = N = 3072 (384): 32.3; 2x8 20.3, 2x4 18.9, 4x8 19.3, 4x4 21.7.           M = 512, K = 12288, N = 3072 (384), rank 128: 63.4; 2x4 45.2, 4x8 43.6
//   M = 512, K = 3072, N = 9216 (1152): 40.5; 2x4 34.0, 4x4 36.9.                       M = 4096, K = 4608, N = 1152 (1152): 59.6; 2x4 51.5, 4x4 54.2
//   M = 2048, K = N = 3072 (1536): 47.6; 2x4 42.9, 4x4 39.6.                            M = 1024, K = 3072, N = 9216 (2304): 59.1; 2x4 53.1, 4x4 52.7
//   M = 4608, K = N = 3072 (3456): 69.5; 2x4 84.9, 4x4 77.0.                            M = 4096, K = 1152, N = 4608 (4608): 47.5; 2x4 55.8, 4x4 51.0
inline int kpar_cols(int variant) { return variant == kKparNarrow ? 32 : 64; }
inline int kpar_rows(int variant) { return variant == kKpar1x8 || variant == kKparNarrow ? 32 : variant == kKpar2x8 || variant == kKpar2x4 ? 64 : 128; }
inline int plan_kpar_int4(int M, int N, int G, int rank, int ksplit_override = 0) {
    if (ksplit_override > 0) return kKparNone;
    const long tn = (N + 63) / 64, t32 = (long)((M + 31) / 32) * tn, t64 = (long)((M + 63) / 64) * tn, t128 = (long)((M + 127) / 128) * tn;
    if (t32 <= 256) return kKpar1x8;
    if (t64 <= 256) return kKpar2x8;
    if (t128 <= 256 && G >= 128) return kKpar4x8;
    // Many tiles of few groups: a round's fixed parts are not earned back, and the 128 x 256 tiles, of which the launch has one or
    // barely two per CU, are faster while the branch is narrow (a wide one makes their activation kernel dear).  Forwards of both
    // kernels over 2300 shapes, us this kernel | 128 x 256 tiles: M = 1024, N = 9216, rank 32: K = 1152 37.6 | 31.2, K = 640 28.6 | 23.5;
    // M = 2048, K = 1536, N = 4608 43.6 | 37.5; M = 1800, K = 1152, N = 4608 36.5 | 32.2; M = 900, K = 320, N = 9216 25.0 | 18.0.  The calls
    // that the last two conditions move gain 13 % in the geometric mean.  Left here: launches that are not wide (M = 4096, K = 1536,
    // N = 2064 36.5 | 40.0; M = N = 3000 37.7 | 42.0), wide branches (M = 1000, K = 1536, N = 9216, rank 128 50.0 | 56.7), and some that
    // lose (M = 1800, K = 2048, N = 4608 49.3 | 43.4).
    if (t64 > 2304 || (t64 > 2048 && G <= 24 && rank <= 32 && N >= 2 * M) || (t64 > 1280 && G <= 5 && rank <= 64)) return kKparNone;
    const long rest = t128 % 512;      // 128-row tiles where their last round of 512 places is at least half full
    return t128 > 256 && (rest == 0 || rest >= 256) ? kKpar4x4 : kKpar2x4;
}

// The INT4 GEMM of a launch that the 128 x 256 tiles do not suit: small tiles whose wavefronts share K, or tiles of 128 x (32 blocks)
// of which a CU holds one (gemm_w4a4_mid_kernel.hip), or neither.
struct SmallInt4 {
    int kpar, blocks;
    int rows() const { return kpar ? kpar_rows(kpar) : blocks ? 128 : 0; }
    int cols() const { return kpar ? kpar_cols(kpar) : 32 * blocks; }
};
// Costs of a launch in units of what one 32 x 32 block costs a CU per group of 64: the tiles of 128 x (32 blocks) by rounds of one
// per CU, the small tiles by their number, the 128 x 256 tiles by rounds of two per CU, of which a last one that gives every CU at most
// one runs at the lone speed.  Fitted to forwards of all three kernels over 85 shapes of more than 480 tiles of 64 x 64, rank 64
// at most (wider branches make partial H dear); the kernel is taken where it comes out 3 % below the others.  us per
// forward, others -> this kernel (blocks; the first two are whole forwards of commit 57cc197 and of 1891fc7 in turn on one box):
//   M = 512, K = 3072, N = 9216 32.6 -> 30.3 (5); M = 4096, K = 4608, N = 1152 49.3 -> 45.4 (5); M = 2048, K = N = 3072 43.7 -> 37.4 (6)
//   M = 609, K = 3712, N = 9360 47.8 -> 41.8 (6); M = 978, K = 4992, N = 9712 87.6 -> 77.0 (5); M = 1774, K = 9536, N = 10256 264 -> 220 (6)
//   M = 2474, K = 1280, N = 1888 24.1 -> 19.7 (5); M = 645, K = 640, N = 6416 19.5 -> 15.3 (5)
// Not beyond four rounds: 35 such launches were 5 % slower (median; M = 1719, K = 4928, N = 14448 163 | 178), 136 of four rounds 2 % faster.
// Without the 3 %: M = 1715, K = 1792, N = 2368 loses 10 %, M = 439, K = 9536, N = 9552 3 %.
inline SmallInt4 plan_small_int4(int M, int N, int G, int rank, int ksplit_override = 0) {
    SmallInt4 s{plan_kpar_int4(M, N, G, rank, ksplit_override), 0};
    const long tm = (M + 127) / 128, t64 = (long)((M + 63) / 64) * ((N + 63) / 64);
    // (not taken, besides: K below 448, which was not measured, and few groups on more tiles than one round of 160 columns, whose second round's
    // fixed parts they do not earn back: M = 4096, K = 1152, N = 4608 47.1 | 48.0)
    if (ksplit_override > 0 || rank > 64 || t64 <= 1024 || G <= 6 || (t64 > 2048 && G <= 25)) return s;
    const long large = tm * ((N + 255) / 256), rest = large % kGemmPlaces;
    double best = s.kpar ? 130 + 1.25 * G * t64 / 256.0
                         : (large / kGemmPlaces + (rest > 256)) * (85 + 2.05 * 8 * G) + (rest > 0 && rest <= 256 ? 85 + 1.1 * 8 * G : 0.0);
    best *= 0.97;
    for (int blocks = 5; blocks <= 6; ++blocks) {
        const long rounds = (tm * ((N + 32 * blocks - 1) / (32 * blocks)) + 255) / 256;
        const double cost = rounds * (125.0 + blocks * G);
        if (rounds <= 4 && cost < best) {
            best = cost;
            s = SmallInt4{kKparNone, blocks};
        }
    }
    return s;
}

// What gemm_w4a4_mid_kernel.hip brings from memory per group for a tile of 128 x (32 blocks) at (gm0, gn0): one-kilobyte pieces, 0 to 6 from
// the tile's four activation blocks, the rest from the weight blocks of 64 columns that cover it wherever it starts.  A piece's uniform
// byte offset counts from the start of the group's blocks.  The last tile of a row may reach past the padded columns: what lies past the
// group's weight blocks (behind the last group: past the buffer) is not asked for, by the rule above (kpar_step).
constexpr int mid_weight_blocks(int blocks) { return (blocks + 1) / 2; }
constexpr int mid_pieces(int blocks) { return (4 * kW4ABlock + mid_weight_blocks(blocks) * kW4BBlock + 1023) / 1024; }
struct MidPiece { int base, lane; };      // uniform offset, lane offset
inline __host__ __device__ MidPiece mid_piece(int j, int lane, int pieces, int gm0, int gn0, int Npad) {
    if (j < 7) return MidPiece{(gm0 / 32) * kW4ABlock + j * 1024, lane * 16};
    const int at = (gn0 / 64) * kW4BBlock + (j - 7) * 1024, end = (Npad / 64) * kW4BBlock;
    return MidPiece{j < pieces && at < end ? at : 0, j < pieces && at + lane * 16 < end ? lane * 16 : (int)0x80000000u};
}

// MXFP4 and INT8 (gemm_kpar_blocks_kernel.hip): one MFMA per block and step and nothing behind it, so these variants are bound
// by what a CU's load unit delivers, (RB + 2) KB for 2 RB MFMAs, and give way to the 128 x 256 tiles, which share their
// operands through LDS, as soon as those fill the CUs.  us per forward, rank 32 / 16, with the large-tile kernels first:
//   M = 1, K = 3072, N = 9216 (144 tiles of 32 x 64): MXFP4 24.8; 1x8 13.2, 2x4 13.7.       INT8 30.3; 1x8 17.3, 2x8 19.3
//   M = 16, K = N = 12288 (192): 38.5; 1x8 24.3, 2x8 26.6.                                   51.6; 1x8 38.2, 2x8 40.8
//   M = 300, K = 3072, N = 2064 (165 of 64 x 64): 28.3; 1x8 19.2, 2x8 15.1, 2x4 14.8.        34.2; 1x8 23.2, 2x8 20.6, 2x4 21.4
//   M = 512, K = N = 3072 (192 of 128 x 64): 26.4; 2x4 18.1, 4x8 17.8, 4x4 18.3.             32.4; 2x4 24.5, 4x8 25.6, 4x4 27.2
//   M = 512, K = 12288, N = 3072 (192): 38.6; 2x4 38.6, 4x8 34.9, 4x4 38.1.                  52.4; 2x4 50.4, 4x8 47.5, 4x4 52.4
//   M = 1024, K = N = 3072 (384): 28.6; 2x4 24.6, 4x8 28.0, 4x4 24.4.                        42.8; 2x4 37.1, 4x8 39.8, 4x4 33.5
//   M = 512, K = 3072, N = 9216 (576): 27.9; 2x4 31.0, 4x4 29.8.                             39.6; 2x4 41.6, 4x4 43.3
//   257 to 512 tiles of 128 x 64, 4x4 | 128 x 128 (or 192 x 128) tiles, each with the activation kernel that goes with it, ranks 16 to 64: MXFP4 M = 1558, K = 1152,
//   N = 1952 15.9 | 12.9; M = 427, K = 2112, N = 4832 17.3 | 15.4; M = 300, K = 3008, N = 8000 20.1 | 17.8; M = 1024, K = N = 3072 18.8 | 18.3; M = 1283, K = 4032, N = 2560 25.3 | 24.3;
//   from K = 4096 on, where the large tiles would split K, M = 600, K = 4096, N = 5632 23.3 | 30.2.  Not taken: rank 128, M = 1100, K = 2624, N = 2880 27.4 | 26.9 (the sums
//   of its cut runs lie in the smaller tiles' workspace), and ranks below 32 beyond K = 1792, which bring few columns of partial H (M = 1800, K = 3328, N = 1536 20.4 | 19.0); K below
//   1024 keeps the small tiles, which lose 1 to 20 % up to K = 512 (MXFP4, M = 500, N = 8000, rank 32 12.0 | 10.6; INT8 13.7 | 12.9) and lie on either side beyond (K = 768, rank 32, MXFP4 M = 500, N = 6400 13.1 | 13.6,
//   M = 1200, N = 2560 13.3 | 11.6, rank 64 15.1 | 16.3; INT8 M = 500, N = 6400 13.3 | 14.8).  INT8 M = 1558, K = 1152, N = 1952 17.2 | 15.1; M = 1476, K = 1024, N = 2432 17.2 | 15.0; M = 1011, K = 1536,
//   N = 2832 16.7 | 16.7.  Nor few tokens, whose runs' partial H these tiles add by themselves while the large ones need a launch for it: MXFP4 up to 240 tokens (M = 16, K = 3072,
//   N = 18432, rank 64 17.5 | 19.4; M = 1, N = 32000, rank 32 17.9 | 19.2; M = 129, K = 1024, N = 16000 14.1 | 15.2; M = 200, K = 1792, N = 12800, rank 16 15.1 | 16.3; M = 256, K = 1792, N = 8640,
//   one pass of eight tokens, 15.5 | 13.6), but ranks 48 and 64 from 97 tokens and K = 1152 on (M = 129, K = 3072, N = 12800, rank 48 20.7 | 19.8; M = 128, K = 1792, N = 25600, rank 64
//   19.2 | 17.8; K = 1024, M = 200, N = 12800 15.6 | 15.9) and no branch at all (M = 1, K = 1152, N = 25600 10.6 | 9.3); INT8 without a branch (M = 500, K = 1152, N = 6400 12.6 | 13.4)
//   and with one of more than 16 columns up to 64 tokens (M = 4, K = 1024, N = 25600, rank 32 13.4 | 14.0; M = 100 15.3 | 14.9)
//   32 x 32 tiles with sixteen wavefronts, 1x8 -> narrow, ranks 16 to 128 (a launch of few tiles pulls its weights through few CUs):
//   INT8: M = 4, K = 10048, N = 1232 (20 tiles of 32 x 64) 18.7 -> 15.8, M = 82, K = 6208, N = 1888 (90) 15.8 -> 14.1, M = 7, K = 1984, N = 4176 (66) 9.4 -> 8.8,
//   M = 3, K = 1408, N = 1584 8.05 -> 8.05; MXFP4: M = 1, K = 5056, N = 1344 13.1 -> 12.3, M = 5, K = 8640, N = 4592 (72) 17.0 -> 15.8, M = 9, K = 2176,
//   N = 4000 10.30 -> 10.32, M = 28, K = 1152, N = 2752 9.8 -> 10.3; beyond 128 tiles of 32 x 64 it loses (INT8, M = 99, K = 9024, N = 2864 19.8 -> 25.9);
//   fewer than 16 were not measured
inline int plan_kpar_blocks(bool i8, int M, int N, int G, int rank, int ksplit_override = 0) {
    if (ksplit_override > 0) return kKparNone;
    const long tn = (N + 63) / 64, t32 = (long)((M + 31) / 32) * tn, t64 = (long)((M + 63) / 64) * tn, t128 = (long)((M + 127) / 128) * tn;
    if (t32 <= 128 && t32 >= 16 && G >= (i8 ? 20 : 52)) return kKparNarrow;
    if (t32 <= 256) return kKpar1x8;
    if (t64 <= 256) return i8 ? kKpar2x8 : kKpar2x4;
    if (t128 <= 256) return i8 && G < 128 ? kKpar2x4 : kKpar4x8;
    const bool few = i8 ? rank == 0 || (rank > 16 && M <= 64) : rank > 0 && M <= (rank >= 48 && G >= 18 ? 96 : 240);
    return t128 <= 512 && (G < 16 || G > (i8 ? 18 : rank < 32 ? 28 : 63) || rank > 64 || few) ? kKpar4x4 : kKparNone;
}

// INT4 and MXFP4 forwards that run as ONE launch (fused_small_kernel.hip): launches of at most one 32 x 64 tile per CU whose K is
// short enough for every tile to quantize its tokens again.  us per forward back to back, two launches | one, rank 32:
//   INT4   M = 1, N = 1152: K = 1024 8.6 | 7.0, 1536 8.8 | 7.9, 1792 9.2 | 8.3, 2048 9.4 | 9.2;  M = 256: K = 1024 9.6 | 7.1, 1792 10.1 | 8.6, 2304 11.1 | 10.2
//          M = 32, N = 16384: K = 1024 9.0 | 7.3, 1792 10.6 | 9.4, 2048 11.4 | 10.9
//   MXFP4  M = 1, N = 1152: K = 1024 9.1 | 6.5, 1792 9.1 | 7.7, 2048 9.2 | 8.3;  M = 256: K = 1024 9.2 | 6.7, 1792 9.1 | 7.9;  M = 8, N = 192: K = 1792 9.2 | 7.6
// In a replayed graph, where no host stands between the launches, the last gain is that of K = 1792 (INT4 4 to 12 %, MXFP4 2 to 9 %;
// K = 2048 2 % slower to 5 % faster, MXFP4 4 % slower to 3 % faster).  Wider branches lose: rank 64, M = 8, K = 1536, N = 9216 9.3 | 11.3.  K below 1024
// keeps its two launches, whose cut has rules of its own (act_short_runs), although one is the faster side there as well (INT4 M = 256, N = 1152: K = 512 8.6 | 6.7, 960 9.6 | 7.5; MXFP4 M = 32,
// N = 16384, K = 960 8.6 | 7.6): the kernel's tests stop at 1024.
inline bool fused_small(int G, int rank, int kpar) { return kpar == kKpar1x8 && rank <= 32 && G >= 16 && G <= 28; }

// How the W4A4 GEMM of an M x N x (64 G) layer is launched.  Tiles are 128 x 256, two workgroups per CU (512 places).
// The K loops of a launch with at most one workgroup per CU can be split over up to eight workgroups per tile (at least
// twelve groups each): every one of them writes its fp32 partial tile to the workspace, and the one that finishes last
// adds them up (in split order, so the result does not depend on who is last) and stores Y.  Left to themselves such
// launches run the kernel whose wavefronts share K instead (plan_kpar_int4) and park nothing; the workspace keeps room
// for the split, which a caller can ask for (SVDQ_OPT_KSPLIT).
// The kernel can also split only the last `tail` tiles of the launch order (the partly filled last round of a large
// launch); measured on the FLUX.1 shapes that gains nothing, because parked tiles travel with device-scope accesses,
// past the L2, at a fraction of the ordinary bandwidth: 1728 tiles with the last 192 split two ways ran 192.9 us
// against 192.2 us unsplit, and every forced split of a large launch was slower.  So large launches are not split.
struct GemmPlan {
    int bm, bn;
    int tiles;       // output tiles
    int tail;        // how many of them (the last in launch order) are split
    int ksplit;      // workgroups per split tile, >= 1; workgroups in all = tiles - tail + tail * ksplit
};
constexpr int kMaxKSplit = 8;
inline GemmPlan plan_gemm(int M, int N, int G, int ksplit_override = 0) {
    GemmPlan pl;
    pl.bm = 128; pl.bn = 256;
    pl.tiles = ((M + 127) / 128) * ((N + 255) / 256);
    int s = 1;
    pl.tail = pl.tiles;
    if (pl.tiles <= kGemmPlaces / 2) {
        s = kGemmPlaces / pl.tiles;
        if (s > kMaxKSplit) s = kMaxKSplit;      // (48 tiles, K = 12288: eight shares 47.6 us, four 50.0, six 52.8)
    }
    while (s > 1 && G / s < 12) --s;                // at least twelve groups per split
    if (ksplit_override > 0) {
        // forced: all tiles of a small launch, the tiles of the last round of a larger one
        s = ksplit_override < kMaxKSplit ? ksplit_override : kMaxKSplit;
        if (pl.tiles > kGemmPlaces / 2) pl.tail = pl.tiles % kGemmPlaces;
    }
    if (s > G) s = G > 0 ? G : 1;
    const int per = (G + s - 1) / s;
    pl.ksplit = (G + per - 1) / per;                // no empty split
    if (pl.ksplit <= 1 || pl.tail == 0) {
        pl.ksplit = 1;
        pl.tail = 0;
    }
    return pl;
}

// LDS bytes of one activation-kernel workgroup with `waves` wavefronts that covers `groups` groups of K: 1 / lambda of
// those channels (fp32), plus one private block per wavefront (X turn-around during the loop, partial H at the end).
constexpr int kLdsBytesPerCU = 160 * 1024;
constexpr int kActOutStage = 2 * 384 + 64;      // a wavefront's 16 tokens of one group on their way out: codes of both halves, scales
inline size_t act_lds_bytes(int groups, int rank, int waves) {
    const int rbmax = rank <= 32 ? 2 : rank <= 64 ? 4 : rank <= 128 ? 8 : 16;
    const size_t red = (size_t)16 * (rbmax * 16 + 1) * 4;
    // (a wavefront works on two groups at a time: two blocks of 16 x 144 bytes of X, two staging blocks)
    return (size_t)groups * kGroup * 4 + (size_t)waves * ((red > 4608 ? red : 4608) + 2 * kActOutStage);
}
// Wavefronts of a workgroup that walks all of K by itself: eight when K gives each of them a few groups and their LDS fits.
inline int act_waves(int K, int rank) { return (K / kGroup >= 32 && act_lds_bytes(K / kGroup, rank, 8) <= (size_t)kLdsBytesPerCU) ? 8 : 4; }

// How the INT4 forward's activation kernel is cut up.  A workgroup owns 16 tokens and a run of `gchunk` groups of K
// (`chunks` runs cover K).  A workgroup's life is a chain of round trips to memory, one per two groups of a wavefront's
// share, so a launch with few 16-token slices, or a long K, is cut into shorter runs that share the CUs; the workgroups
// of a slice then park their partial H in the workspace and the last one to arrive adds them up in run order.  Parked
// sums travel with device-scope accesses, past the L2, and cost more than they look: the runs are cut only as far as
// the launch needs to reach two to three workgroups per CU.
constexpr int kActChunkWhole = 255;      // override value: one run, all of K
inline ActPlan plan_act(int M, int G, int rank, int gchunk_override = 0) {
    ActPlan pl;
    const int slices = (M + 15) / 16;
    // Measured on the FLUX.1 / PixArt shapes.  A launch with more slices than CUs walks K whole, up to 192 groups (48 KB
    // of smoothing factors in LDS, two workgroups per CU): at M = 4608, K = 12288 whole slices take 45.9 us (rank 32) and
    // 72.8 us (rank 128), runs of 96 groups 46.4 and 75.0, runs of 48 groups 52.0 and 83.3.  A launch with a
    // workgroup for every other CU at least is left alone up to K = 4608 and cut into runs of 48 groups beyond; a
    // launch with fewer slices is cut into up to eight runs of at least eight groups, towards one workgroup per CU.
    int runs = 1;
    if (slices > 256) runs = (G + 191) / 192;
    else if (slices > 128) runs = G >= 128 ? (G + 47) / 48 : 1;
    else runs = 256 / slices < 8 ? (256 + slices - 1) / slices : 8;
    int gc = (G + runs - 1) / runs;
    if (gc < 8) gc = 8;
    gc = (gc + 3) / 4 * 4;                               // whole groups for each of four wavefronts
    if (gchunk_override > 0) gc = gchunk_override;
    if (gc >= kActChunkWhole || gc > G) gc = G > 0 ? G : 1;
    if ((G + gc - 1) / gc > 64) gc = (G + 63) / 64;      // one arrival word per run and lane
    pl.chunks = (G + gc - 1) / gc;
    if (pl.chunks < 1) pl.chunks = 1;
    pl.gchunk = gc;
    // eight wavefronts when a run gives each of them a few groups and their LDS fits - but a launch with more slices
    // than CUs puts several workgroups on a CU anyway, and those of four wavefronts then share it better
    // (measured at K = 3072: M = 12288 32.6 us against 34.6, M = 16384 41.7 against 44.6; at M = 4608, K = 12288:
    // 45.9 against 49.1, rank 128 72.8 against 78.6)
    pl.waves = (gc >= 32 && act_lds_bytes(gc, rank, 8) <= (size_t)kLdsBytesPerCU) ? 8 : 4;
    if (slices > 256) pl.waves = 4;
    // A launch whose workgroups are 256 q + r leaves r CUs with one workgroup more than the rest, and they set the
    // kernel's time.  Up to r = 128 the slices those r workgroups belong to (the last ones) are cut into shorter runs
    // instead, about 256 workgroups of them, so that every CU gets the same extra share; the other slices stay as they
    // are and pay nothing more for parked sums
    // (measured at K = 3072, rank 32: M = 4608 20.2 -> 16.9 us, 5120 20.5 -> 18.1, 6144 21.4 -> 19.4, 8704 30.1 -> 26.4,
    // 16896 47.2 -> 43.8; rank 128 at M = 4608: 30.1 -> 23.0; with r > 128 a finer cut does not pay).
    pl.whole = 0; pl.chunks0 = 1; pl.gchunk0 = G > 0 ? G : 1;
    pl.deposit = false;
    int twos = 1;                                        // largest power of two that divides the runs per slice (up to 256)
    while (twos < 256 && pl.chunks % (2 * twos) == 0) twos *= 2;
    const int tail = slices % (256 / twos);              // the slices behind the last full round of 256 workgroups
    const int rest = tail * pl.chunks;                   // their workgroups
    if (gchunk_override == 0 && slices > 128 && slices > tail && rest > 0 && rest <= 128 && G >= 16) {
        int c = 256 / rest;
        if (c > 8) c = 8;
        int g2 = (gc + c - 1) / c;
        if (g2 < 4) g2 = 4;
        g2 = (g2 + 3) / 4 * 4;                           // whole groups for each of four wavefronts
        if (g2 < gc && (G + g2 - 1) / g2 <= 64) {
            pl.whole = slices - tail;
            pl.chunks0 = pl.chunks; pl.gchunk0 = gc;
            pl.gchunk = g2;
            pl.chunks = (G + g2 - 1) / g2;
        }
    }
    return pl;
}
// The same where the GEMM is a small-launch kernel (its tile; 0 x 0: it is not).  Such a GEMM can add the
// runs' partial H itself when it loads them, which takes the meeting of a slice's runs - four round trips past the L2 - out of
// the activation kernel; runs then cost next to nothing and are cut so that a wavefront walks three groups.  What they do
// cost is that every tile reads its rows of all partial H: up to 64 MB of that per launch (measured: 50 MB gains 2-3 us,
// 75 MB nothing, 201 MB loses 5), and 512 workgroups.  us per forward, meeting -> deposit (wavefronts, groups per run):
//   K = N = 3072, rank 32: M = 512 20.6 -> 18.4 (4, 12), 18.6 (8, 16), 19.1 (8, 24); M = 1024 29.5 -> 27.4 (4, 12); M = 2048 43.5 -> 40.2 (4, 12)
//   M = 64, K = 12288, N = 3072: 22.1 -> 20.0 (4, 12), 19.8 (8, 24); M = 512 41.7 -> 39.7 (4, 12), 37.6 (8, 24); M = 256, K = N = 1152 12.2 -> 10.3 (4, 12)
//   rank 128, K = N = 3072: M = 64 17.8 -> 14.1 (4, 12), M = 512 26.3 -> 24.3;  M = 512, K = 12288: 48.4 -> 54.1 (201 MB: not taken)
// The 128-row tiles of more than 64 columns make every lane add up its rows' parts between the loads of L2: up to 128 columns of them in all
// runs, beyond that H comes ready-made.  us per forward, added | ready-made: M = 562, K = 3136, N = 9024, rank 64 (5 runs) 47.5 | 39.0, M = 832, K = 3904,
// N = 5408, rank 64 (6) 53.4 | 40.7, M = 396, K = 9792, N = 11584, rank 64 (7) 94.0 | 82.5; 467 launches beyond the line: median 8 % faster, none slower.  In a second and third round the same rows are added up again:
// 96 and 64 columns there.
constexpr int kMidPartColumns = 128;
// fine: shorter runs where the launch does not fill the CUs (act_short_runs); there are more of them, and act_use_small_plan may have to
// take the longer ones.
inline ActPlan plan_act_small(int M, int N, int G, int rank, int act_override, int tile_rows, int tile_cols, bool fine) {
    const ActPlan old = plan_act(M, G, rank, act_override);
    if (act_override > 0 || tile_rows == 0 || rank <= 0 || rank > 128) return old;
    const long slices = (M + 15) / 16;
    ActPlan pl = old;
    // Two groups to a wavefront while that fills the CUs once (three for a narrow branch with a long K, and where wide tiles add the
    // runs for fewer columns): us per forward, 12 or 24 groups per run -> 8: M = 2, K = 1600, N = 7968, rank 128 12.0 -> 10.7; M = 10, K = 10944, N = 9680,
    // rank 128 27.8 -> 21.3; M = 13, K = 1664, N = 6448, rank 64 10.5 -> 9.6; M = 5, K = 6976, N = 10400, rank 32 16.1 -> 15.3; rank 32, M = 16, K = 10240, N = 1728
    // 15.9 -> 16.3 (12: 15.7); M = 390, K = 7424, N = 1184 (375 workgroups) 19.0 -> 20.0
    pl.waves = 4;
    pl.gchunk = tile_cols > 64 || (rank <= 32 && G > 144) ? 12 : 8;
    if (!fine || slices * ((G + 7) / 8) > 256) {
        pl.waves = G > 96 ? 8 : 4;
        pl.gchunk = G > 96 ? 24 : 12;
    }
    if (pl.gchunk > G) pl.gchunk = G;
    pl.chunks = (G + pl.gchunk - 1) / pl.gchunk;
    pl.whole = 0; pl.chunks0 = 1; pl.gchunk0 = G;
    pl.deposit = pl.chunks > 1;
    const long tiles = (long)((M + tile_rows - 1) / tile_rows) * ((N + tile_cols - 1) / tile_cols);
    if (tile_cols > 64 && pl.chunks * rank > (tiles <= 256 ? kMidPartColumns : kMidPartColumns * 3 / 2 / ((tiles + 255) / 256))) return old;
    if (slices * pl.chunks > 512 || pl.chunks > 64 || tiles * tile_rows * rank * 4 * pl.chunks > 64l << 20) return old;
    return pl;
}
// INT4 and MXFP4 launches of wide branches that take the kernel of 64-token workgroups (act_wide_kernel.hip): the number of runs that K
// is cut into (0: they do not), for `room` runs' partial H: up to two workgroups per CU, at least six groups to a run.
// us per forward at rank 128, act_kernel.hip -> this: INT4 M = 4608, K = 12288, N = 3072 247 -> 230, M = 1096, K = 9728, N = 1184 63.4 -> 45.8, M = 780, K = 11520,
// N = 8240 127 -> 117, M = 2595, K = 5632, N = 5136 121.5 -> 114.4; MXFP4 M = 1432, K = 9856, N = 2720 84.9 -> 61.6, M = 1415, K = 6144, N = 2256 59.8 -> 46.3,
// M = 1386, K = 2752, N = 5376 41.0 -> 36.2.  Not taken: few tokens (M = 512, K = 12288, N = 3072 43.9 | 45.1; M = 482, K = 6784, N = 7920 49.3 | 49.9), which 16-token
// workgroups spread further; many tokens with a short K (M = 4608, K = 3072, N = 12288 215 | 218; M = 4539, K = 3520, N = 9408 210 | 215), whose sum launch
// is not earned back.  At rank 64 (half the fragments) M = 4608, K = N = 3072 72.8 | 74.6.
// Few workgroups with long runs, where a layer of few columns or the static workspace has room for few runs only, leave CUs idle: a run of n
// groups takes its workgroup n x 1.1 us (MXFP4 M = 2595, K = 2560, N = 272 26.6 | 44.3; INT4, static, M = 3019, K = 7488, N = 304, rank 112 51.6 | 134.7).
// INT4's other kernel is the faster one of the two formats', and how good it is depends on its own plan (`other`).  Runs on eight wavefronts are slow
// (M = 1445, K = 5440, N = 416, rank 112 39.7 | 30.1), and so are seven or more groups to a wavefront on more than one round of workgroups (M = 2419, K = 4160,
// N = 304, rank 96 34.2 | 29.4, M = 1579, K = 5312, N = 448 35.7 | 31.0); fewer lose to an even load only (M = 2790, K = 2624, N = 400, rank 96, 308 workgroups, a
// second one on a few of the CUs 28.7 | 30.8; M = 577, K = 2752, N = 2576, 80 workgroups 24.1 | 25.9; M = 622, K = 6144, N = 4576, rank 80 42.0 | 44.1).
// The lines are those between faster and slower of 3100 forwards: of those taken 1 in 150 is slower, by 2 to 6 %.
constexpr int kActWideTokens = 64;
inline int plan_act_wide(bool int4, const ActPlan &other, int M, int G, int rank, size_t room) {
    if (rank <= 64 || rank > 128 || M < 576 || G < 40 || (M > 3000 && G < 72)) return 0;
    const int tiles = (M + kActWideTokens - 1) / kActWideTokens;
    size_t runs = tiles < 512 ? 512 / tiles : 1;
    if (runs > (size_t)((G + 5) / 6)) runs = (G + 5) / 6;
    if (runs > room) runs = room;
    if (runs < 1) return 0;
    const int gc = (G + (int)runs - 1) / (int)runs, cut = (G + gc - 1) / gc, workgroups = tiles * cut;
    if (!int4) return gc <= 12 || workgroups >= 144 ? cut : 0;
    const int slices = (M + 15) / 16, other_runs = other.whole > 0 ? other.chunks0 : other.chunks, other_groups = other.whole > 0 ? other.gchunk0 : other.gchunk;
    bool take;
    if (other_runs > 1 && other.waves == 8) take = workgroups >= (gc > 24 ? 176 : 128);
    else if (other_groups > 6 * other.waves && (other_runs == 1 || slices * other_runs > 256)) take = workgroups >= (gc > 12 ? 352 : 128);
    else take = other_runs > 1 && gc <= 12 && M >= 768 && workgroups >= 128 && workgroups <= 256;
    return take ? cut : 0;
}

// INT4 and MXFP4 launches that take the kernel of 32-token workgroups (act_tile_kernel.hip): the number of runs that K is cut into (0: they do not),
// for `room` runs' partial H.  `other`: the plan of the 16-token workgroups, which do not leave partial H for the GEMM.  Two workgroups per CU up
// to rank 64, one beyond; the number of runs is that of whole rounds of the four wavefronts, two of them at least and three of a K above 64 groups, and K is then cut into so
// many runs of about one length (33 groups: four of seven and one of five).
// us per forward, act_kernel.hip | this, ranks above 32: INT4 M = 1440, K = 1792, N = 2336, rank 128 31.9 | 25.2; M = 1255, K = 9856, N = 528, rank 48 37.0 | 29.6; M = 512,
// K = 12288, N = 3072, rank 128 42.7 | 39.7; M = 320 35.6 | 28.9; M = 913, K = 10624, N = 5984, rank 64 93.6 | 85.0; MXFP4 M = 131, K = 10688, N = 4352, rank 128 29.2 | 23.8; M = 3078,
// K = 2368, N = 1936, rank 128 36.4 | 32.6.  Not taken: more than 2048 tokens, which fill the CUs with 16 to a workgroup, with a short K (INT4 M = 3246, K = 1408, N = 432,
// rank 64 17.0 | 19.5; M = 4006, K = 2816, N = 2736, rank 64 60.6 | 62.8; MXFP4 M = 2235, K = 1664, N = 768, rank 96 19.7 | 20.8).
// Up to rank 32 only where the runs of the other kernel meet: M = 1500, K = 8192, N = 2048, rank 16 51.7 | 45.8, M = 2300, K = 9216, rank 32 75.8 | 70.8; else
// M = 3000, K = 6144, N = 3072, rank 16 95.2 | 96, MXFP4 M = 1500, K = 3072, N = 4608 28.3 | 28.9 (one pass); and from 257 tokens on (below, the sum's launch is the larger part: MXFP4 M = 128,
// K = 1024, N = 36864, rank 16 15.5 | 16.7, M = 171, K = 8192, N = 23408 36.0 | 37.9, INT4 M = 256, K = 1024, N = 36864 27.6 | 28.5, M = 64, K = 8192, N = 23408, rank 32 40.8 | 41.4; INT4 M = 400,
// K = 4096, N = 23408, rank 32 66.1 | 66.3).  Ranks of 48 and 64 give way to one pass with
// eight tokens to a workgroup where that is taken (MXFP4 up to K = 3072): M = 2048, K = N = 3072, rank 64 29.5 | 28.0; M = 1024, K = 1536, N = 9216, rank 48 25.5 | 23.6.
constexpr int kActTileTokens = 32;
inline int plan_act_tile(const ActPlan &other, bool one_pass, int M, int G, int rank, size_t room) {
    if (rank > 128 || G < 16 || M > 4096) return 0;
    if (rank <= 64 && one_pass && M <= 2048) return 0;
    if (rank <= 32 && (M <= 256 || one_pass || other.chunks <= 1 || other.whole != 0)) return 0;
    if (rank > 32 && M > 2048 && G < (rank > 64 ? 36 : 72)) return 0;
    const int tiles = (M + kActTileTokens - 1) / kActTileTokens;
    size_t runs = (rank > 64 ? 256 : 512) / tiles;
    if (runs > room) runs = room;
    if (runs < 1) return 0;
    int gc = (G + (int)runs - 1) / (int)runs;
    gc = (gc + 3) / 4 * 4;
    if (gc < (G > 64 ? 12 : 8)) gc = G > 64 ? 12 : 8;
    const int cut = (G + gc - 1) / gc;
    return gc <= 12 || tiles * cut >= 128 ? cut : 0;
}

// Where partial H is left for the GEMM, H itself is never made in memory; its first 16 bytes name the place of the parts instead, for
// svdq_debug_act: two words that no sum of products gives (a NaN with this payload), the number of runs, and how many 256-byte
// units behind H the parts [runs][Mpad][rank] start.
constexpr uint32_t kHInParts0 = 0x7fc5eed1u, kHInParts1 = 0x7fd0e571u;
// the value a workgroup leaves in its arrival word; the word is cleared again before the kernel ends, so whatever a
// fresh workspace holds is taken for "not arrived" (anything but this one 64-bit value)
constexpr unsigned long long kActArrived = 0x5356445141525256ull;
// what the cut slices of a launch park in the workspace: fp32 partial H of every run, and one arrival word per run
inline size_t act_parked_floats(const ActPlan &a, int Mpad, int rank) {
    return (a.whole > 0 && a.chunks0 > 1 ? (size_t)a.chunks0 * 16 * a.whole * rank : 0) + (a.chunks > 1 ? (size_t)a.chunks * (Mpad - 16 * a.whole) * rank : 0);
}
inline size_t act_arrival_words(const ActPlan &a, int Mpad) {
    return (a.whole > 0 && a.chunks0 > 1 ? (size_t)a.chunks0 * a.whole : 0) + (a.chunks > 1 ? (size_t)a.chunks * (Mpad / 16 - a.whole) : 0);
}

// A K of 9 to 12 groups is one long run, whose H the activation kernel makes by itself, or two short ones that every tile adds.  us per forward,
// one run | two: MXFP4 32-row tiles 4 to 12 % faster in two (M = 136, K = 640, N = 9248, rank 96 on 128-row tiles 15.1 | 17.3, M = 713, K = 576,
// N = 1408, rank 32 11.5 | 12.3); INT4 32-row tiles at ranks from 48 on 3 to 5 % faster, narrower ones 9.4 | 9.6 (M = 6, K = 576, N = 7136), taller tiles
// M = 365, K = 640, N = 6016, rank 96 16.5 | 19.3, M = 986, K = 704, N = 6544, rank 32 21.9 | 23.6.
inline bool act_short_runs(bool int4, int G, int rank, int tile_rows) { return G > 12 || (int4 ? tile_rows <= 32 && rank >= 48 : tile_rows <= 64); }
// Gives a workspace a plan of plan_act_small where what that plan parks fits into what the workspace holds from
// partial_off on: the launches it is made for leave the room of the GEMM's partial tiles unused, and
// a workspace's size stays what callers may have kept from the plan above.
template <typename W>
inline bool act_plan_fits(W &w, const ActPlan &a, int rank) {
    const bool parked = a.chunks > 1 && rank > 0;
    const size_t h = parked ? align256(act_parked_floats(a, w.Mpad, rank) * 4) : 0, words = parked ? align256(act_arrival_words(a, w.Mpad) * 8) : 0;
    if (a.chunks > 1 && !a.deposit) return false;
    if (w.partial_off + h + words > w.total) return false;
    w.act = a;
    w.hpart_off = w.partial_off;
    w.aflags_off = w.hpart_off + h;
    return true;
}
// Where the short runs are too many, for the workspace of a layer of few columns or for the tiles to read, longer ones whose partial H the
// GEMM adds too, or the meeting: us per forward, meeting | longer runs: MXFP4 M = 4, K = 5312, N = 512, rank 128 18.7 | 13.4, M = 128, K = 5888, N = 128
// 19.6 | 16.1; INT4 M = 119, K = 5184, N = 7712, rank 128 24.4 | 21.4, M = 2, K = 13568, N = 128, rank 96 25.3 | 23.3.  Not taken: K above 6144 beyond one
// slice (MXFP4 M = 69, K = 7296, N = 6304, rank 112 22.9 | 28.0), more tokens or 128-row tiles (INT4 M = 323, K = 3904, N = 5824, rank 64 28.8 | 32.2).
inline bool act_longer_runs(int M, int G, int tile_rows) { return tile_rows > 0 && tile_rows <= 64 && M <= (G <= 96 ? 256 : 16); }
// INT4 and MXFP4 launches that leave no partial H although their tiles could add it: one pass with eight tokens to a workgroup makes H itself in
// about the time, and the tiles are spared its reading.  us per forward, partial H | one pass: INT4 M = 1024, K = 1152, N = 4608 22.0 | 18.6; M = 1590, K = 1792, N = 2848
// 26.7 | 22.3; M = 2048, K = N = 3072 37.4 | 34.7; M = 521, K = 1728, N = 1424 12.3 | 11.7; MXFP4 M = 1024, K = 2048,
// N = 1536 14.1 | 13.2; M = 512, K = N = 3072 16.0 | 15.5.  With three groups to a wavefront up to 1024 tokens, which the runs' workgroups take in one round, not for INT4 (M = 512, K =
// N = 3072 16.8 | 17.9, on 128 x 160 tiles N = 9216 31.1 | 30.1; M = 1024, K = 3072, N = 1536 16.9 | 18.2, N = 4096 25.7 | 26.1, but N = 4608 30.9 | 29.6 and K = 2112, N = 4608 26.5 | 24.0), and for MXFP4 not on tiles of 32 or 64 rows, which are few and read
// little (M = 371, K = 2560, N = 256 9.9 | 10.6, M = 512, K = 2560, N = 1024 11.0 | 11.5, M = 1024, K = 3072, N = 1024 13.3 | 14.1; tiles of 128 rows M = 771, N = 1536 7 and 2 % faster at K = 2560 and 3072).
// Nor MXFP4 with 16 columns of H (wider branches were not measured).  Fewer tokens and groups keep partial H; on the far sides, partial H | one pass: M = 300, K = 1024, N = 3072 INT4 10.9 | 10.2, MXFP4 10.1 | 10.0;
// M = 340, K = 2048 INT4 14.2 | 14.0, MXFP4 13.6 | 12.6; M = 256, K = 3072, N = 1152 INT4 12.8 | 13.0, MXFP4 11.2 | 11.3; M = 1000, N = 3072: K = 896 INT4 16.3 | 15.2, MXFP4 14.5 | 13.6, K = 512 INT4 13.8 | 13.5, MXFP4
// 12.3 | 12.3, K = 256 INT4 11.5 | 11.8, MXFP4 11.5 | 12.0.
inline bool act_pass_instead(bool int4, int M, int N, int G, int rank, int tile_rows) {
    if (M <= 368 || M > 2048 || G < 16 || G > 48 || rank > 32) return false;
    return int4 ? rank > 0 && (G <= 32 || M > 1024 || (M == 1024 && (G <= 40 || N > 4096))) : rank > 16 && (G <= 32 || M > 1024 || tile_rows > 64);
}
template <typename W>
inline void act_use_small_plan(W &w, bool int4, int M, int N, int G, int rank, int act_override, int tile_rows, int tile_cols) {
    if (act_override == 0 && act_pass_instead(int4, M, N, G, rank, tile_rows)) return;
    const bool fine = act_short_runs(int4, G, rank, tile_rows);
    if (act_plan_fits(w, plan_act_small(M, N, G, rank, act_override, tile_rows, tile_cols, fine), rank)) return;
    if (fine && act_longer_runs(M, G, tile_rows)) act_plan_fits(w, plan_act_small(M, N, G, rank, act_override, tile_rows, tile_cols, false), rank);
}

// INT8 batches that act_w8_small_kernel.hip takes, of those whose plan cuts K (at most 128 slices): where the GEMM adds the runs'
// partial H itself (kpar); where a launch of its own has to, rows that one pass does not take or takes slower.  us per forward, walking or one-pass
// kernel -> this one: M = 1, K = 3648, N = 5200 17.5 -> 11.3; M = 14, K = 5760, N = 1568 22.5 -> 13.8; M = 4, K = 10048, N = 1232 24.7 -> 18.7;
// M = 3, K = 1408, N = 1584 10.6 -> 8.1; M = 664, K = 6976, N = 1824 39.7 -> 30.7; M = 1293, K = 6016, N = 1616 45.7 -> 39.5; with the launch: M = 1104, K = 7424, N = 9408
// 108 -> 97.  Where H is added by a launch of its own, one pass with eight tokens to a workgroup is the faster one (this kernel | one pass) up to K = 3072:
// M = 270, K = 1152, N = 12288 18.8 | 17.4; M = 620, K = 2816, N = 11488 33.3 | 32.2; M = 1, K = 3072, N = 36864 28.8 | 28.7; and up to K = 6144 from 1153 tokens on: M = 1700,
// K = 4096, N = 8192 73.8 | 70.6; M = 1337, K = 6144, N = 4096 50.3 | 49.1; below, M = 270, K = 6144, N = 12288 41.6 | 42.9, M = 594, K = 3776, N = 6896 32.3 | 32.7,
// M = 893, K = 4224, N = 4928 34.4 | 34.3, M = 1000, K = N = 4608 41.7 | 40.3.  Few tokens of a K below 1024 keep this kernel, slower by 6 to 11 %
// there too (M = 16, K = 640, N = 36864 13.9 | 12.8, M = 400, K = 960, N = 9216 17.2 | 15.7), and so do two kinds of launches that one pass is slower for: without
// a branch, where nothing has to be added (M = 16, K = 2048, N = 39936 20.3 | 21.5, M = 512, K = 1536, N = 9984 17.9 | 18.7, M = 400, K = 3072, N = 9984 26.1 | 27.4), and up to 256 tokens of a K above 2560 with more
// than 16 columns of H (M = 4, K = 3072, N = 33024, rank 32 28.1 | 29.3, rank 16 27.4 | 27.5; M = 200, N = 19968 30.5 | 31.0; M = 400, N = 9984 30.2 | 30.4).
inline bool act_w8_small(int M, int K, int rank, int kpar) {
    const int G = K / kGroup, slices = (M + 15) / 16;
    return G <= 192 && rank <= 32 && (kpar || G > 96 || (G > 48 && slices <= 72) || ((G < 16 || rank == 0) && slices <= 48) || (rank > 16 && G > 40 && slices <= 16));
}

// The int8 MFMA takes twice the time of the 4-bit one per step of 64 channels, so a split of the 8-bit GEMM's K loop pays
// from sixteen such steps per share on (measured at M = 512: K = 3072, 48 tiles: 28.0 -> 23.2 us with three shares;
// K = 4608, 20 tiles: 39.8 -> 28.2 us with four; K = 12288, 48 tiles: 83.5 -> 39.5 us with four).
constexpr int kW8MinSplitSteps = 16;
// Workspace of the 8-bit forward: int8 codes in operand order, one fp16 scale per token, H twice (fp32 and bf16 parts),
// and for small launches with a long K the arrival counters and int32 partial tiles of a split K loop (the MXFP4
// GEMM's plan: same tiles, same rule).
struct WorkspaceW8 {
    size_t codes_off, sx_off, h_off, hfrag_off, counters_off, partial_off, pmax_off, hpart_off, aflags_off, total;
    int Mpad;
    int n_counters, ksplit;
    bool act_cut;      // the activation kernel runs twice over K cut into runs (small launches): maxima of the runs, then the rest
    ActPlan act;
};
inline WorkspaceW8 workspace_layout_w8(int M, int K, int N, int rank, int ksplit_override = 0, int act_override = 0) {
    WorkspaceW8 w;
    w.Mpad = round_up(M > 0 ? M : 1, kRowPad);
    w.codes_off = 0;
    w.sx_off = align256((size_t)K * w.Mpad);
    w.h_off = w.sx_off + align256((size_t)w.Mpad * 2);
    w.hfrag_off = w.h_off + align256((size_t)w.Mpad * (rank > 0 ? rank : 1) * 4);
    w.counters_off = w.hfrag_off + align256((size_t)w.Mpad * (rank > 0 ? rank : 1) * 4);
    const GemmPlanFp4 pl = plan_gemm_fp4(M > 0 ? M : 1, N, K / kGroup, ksplit_override, kW8MinSplitSteps);
    w.ksplit = pl.ksplit;
    w.n_counters = pl.ksplit > 1 ? pl.tiles : 0;
    w.partial_off = w.counters_off + align256((size_t)w.n_counters * 4);
    w.pmax_off = w.partial_off + (pl.ksplit > 1 ? align256((size_t)pl.ksplit * pl.tiles * 128 * 256 * 4) : 0);
    // A token's scale needs its maximum over all of K, so the one-pass kernel gives a slice to one workgroup; a launch
    // with few slices runs two passes over a cut K instead, like the INT4 forward's (measured at M = 512, K = 12288:
    // 44 us in one pass)
    w.act = plan_act(M > 0 ? M : 1, K / kGroup, rank, act_override);
    w.act_cut = w.act.chunks > 1 && w.act.whole == 0 && (M + 15) / 16 <= 128;
    w.hpart_off = w.pmax_off + (w.act_cut ? align256((size_t)w.act.chunks * w.Mpad * 4) : 0);
    const bool parked = w.act_cut && rank > 0;
    w.aflags_off = w.hpart_off + (parked ? align256(act_parked_floats(w.act, w.Mpad, rank) * 4) : 0);
    w.total = w.aflags_off + (parked ? align256(act_arrival_words(w.act, w.Mpad) * 8) : 0);
    return w;
}

// Workspace of the MXFP4 forward (WorkspaceFp4 above).
inline WorkspaceFp4 workspace_layout_fp4(int M, int K, int N, int rank, int ksplit_override = 0, int act_override = 0) {
    WorkspaceFp4 w;
    w.Mpad = round_up(M > 0 ? M : 1, kRowPad);
    const int G = K / kGroup;
    w.codes_off = 0;
    w.bx_off = align256((size_t)G * w.Mpad * kFp4RowBytes);
    w.h_off = w.bx_off + align256(fp4_scale_bytes(G, w.Mpad));
    w.hfrag_off = w.h_off + align256((size_t)w.Mpad * (rank > 0 ? rank : 1) * 4);
    w.counters_off = w.hfrag_off + align256((size_t)w.Mpad * (rank > 0 ? rank : 1) * 4);
    const GemmPlanFp4 pl = plan_gemm_fp4(M > 0 ? M : 1, N, G, ksplit_override);
    w.n_counters = pl.ksplit > 1 ? pl.tiles : 0;
    w.partial_off = w.counters_off + align256((size_t)w.n_counters * 4);
    w.hpart_off = w.partial_off + (pl.ksplit > 1 ? align256((size_t)pl.ksplit * pl.tiles * 128 * 256 * 4) : 0);
    // the activation kernel's partial H [chunks][rows of the cut slices][rank] fp32 and one arrival word per workgroup, as in the INT4 workspace
    const ActPlan ap = plan_act(M > 0 ? M : 1, G, rank, act_override);
    w.act = ap;
    const bool parked = ap.chunks > 1 && rank > 0;
    w.aflags_off = w.hpart_off + (parked ? align256(act_parked_floats(ap, w.Mpad, rank) * 4) : 0);
    w.total = w.aflags_off + (parked ? align256(act_arrival_words(ap, w.Mpad) * 8) : 0);
    const int kpar = plan_kpar_blocks(false, M > 0 ? M : 1, N, G, rank, ksplit_override);
    act_use_small_plan(w, false, M > 0 ? M : 1, N, G, rank, act_override, kpar ? kpar_rows(kpar) : 0, kpar ? kpar_cols(kpar) : 0);
    return w;
}

// Workspace carve-up for a forward of M tokens.
struct Workspace {
    size_t codes_off, h_off, hfrag_off, counters_off, partial_off, hpart_off, aflags_off, total;
    int Mpad;
    int n_counters;      // one arrival counter per tile whose K loop is split
    ActPlan act;
};
// lean: a launch that runs the kernel whose wavefronts share K gets no room for a split K loop, which it does not make, and all
// the room it needs for the partial H that its GEMM adds (the static workspace, whose size is given; the public size stays as it was).
inline Workspace workspace_layout(int M, int K, int N, int rank, int ksplit_override = 0, int act_override = 0, bool lean = false) {
    Workspace w;
    w.Mpad = round_up(M > 0 ? M : 1, kRowPad);
    const int G = K / kGroup;
    w.codes_off = 0;                                                     // activation blocks: codes and scales
    w.h_off = align256(w4_a_bytes(G, w.Mpad));
    w.hfrag_off = w.h_off + align256((size_t)w.Mpad * (rank > 0 ? rank : 1) * 4);
    w.counters_off = w.hfrag_off + align256((size_t)w.Mpad * (rank > 0 ? rank : 1) * 4);
    const GemmPlan pl = plan_gemm(M > 0 ? M : 1, N, G, ksplit_override);
    const SmallInt4 sm = plan_small_int4(M > 0 ? M : 1, N, G, rank, ksplit_override);
    const bool no_split = lean && sm.rows() > 0;
    w.n_counters = no_split ? 0 : pl.tail;                                // one arrival counter per split tile
    w.partial_off = w.counters_off + align256((size_t)w.n_counters * 4);
    w.hpart_off = w.partial_off + (no_split ? 0 : align256((size_t)pl.ksplit * pl.tail * pl.bm * pl.bn * 4));
    // the activation kernel's partial H [chunks][rows of the cut slices][rank] fp32 and one arrival word per workgroup
    w.act = plan_act(M > 0 ? M : 1, G, rank, act_override);
    const bool parked = w.act.chunks > 1 && rank > 0;
    w.aflags_off = w.hpart_off + (parked ? align256(act_parked_floats(w.act, w.Mpad, rank) * 4) : 0);
    w.total = w.aflags_off + (parked ? align256(act_arrival_words(w.act, w.Mpad) * 8) : 0);
    const bool fine = act_short_runs(true, G, rank, sm.rows());
    ActPlan small = plan_act_small(M > 0 ? M : 1, N, G, rank, act_override, sm.rows(), sm.cols(), fine);
    if (fine && !small.deposit && small.chunks > 1 && act_longer_runs(M > 0 ? M : 1, G, sm.rows())) small = plan_act_small(M > 0 ? M : 1, N, G, rank, act_override, sm.rows(), sm.cols(), false);
    if (no_split && small.deposit) {
        const size_t need = w.partial_off + align256(act_parked_floats(small, w.Mpad, rank) * 4) + align256(act_arrival_words(small, w.Mpad) * 8);
        if (w.total < need) w.total = need;
    }
    act_use_small_plan(w, true, M > 0 ? M : 1, N, G, rank, act_override, sm.rows(), sm.cols());
    return w;
}

}  // namespace svdq
