"""What the forwards ask of the HIP runtime, recorded on the CPU (host_launch_recorder.cpp): the host half of every launch
runs as it is, nothing reaches a GPU."""
import os
import shutil
import subprocess

import pytest

from paper_2411_05007_amd import svdq as S
from tests import test_gpu_small_launches as G
from tests.test_gpu_canaries import KERNELS as G_CANARIES

HERE = os.path.dirname(os.path.abspath(__file__))
INT4, STATIC, FP4, W8A8, W4A16 = 64, 65, 32, 0, 16


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    if not os.path.exists(S.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    exe = str(tmp_path_factory.mktemp("rec") / "recorder")
    subprocess.run([cxx, "-std=c++17", "-O1", "-rdynamic", os.path.join(HERE, "host_launch_recorder.cpp"), "-o", exe, "-ldl"], check=True)

    def run(calls):
        """One list of records per call (device, format, M, K, N, rank[, options[, output]]); all calls in one process."""
        text = "".join(" ".join(str(v) for v in (*c, 0, 0)[:8]) + "\n" for c in calls)
        r = subprocess.run([exe, S.LIB_PATH], input=text, capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr
        out, cur = [], []
        for line in r.stdout.splitlines():
            w = line.split()
            if w[0] == "status":
                assert w[1] == "0", (calls[len(out)], w)
                out.append(cur)
                cur = []
            else:
                cur.append((w[0], int(w[1]), w[2], *(int(v) for v in w[3:])))
        assert len(out) == len(calls)
        return out
    return run


# one call for every kernel family: K-sharing and large tiles, one-pass and walking activation kernels, forced splits
SHAPES = [(INT4, 256, 1152, 1152, 32), (INT4, 512, 12288, 3072, 128), (INT4, 4608, 3072, 12288, 32), (INT4, 4096, 4608, 1152, 32), (INT4, 512, 3072, 3072, 32, 3 << 8),
          (FP4, 512, 3072, 3072, 32), (FP4, 4608, 3072, 12288, 32), (FP4, 1337, 3072, 9216, 32), (FP4, 100, 6144, 272, 32, 3 << 8),
          (W8A8, 1337, 3072, 9216, 16), (W8A8, 512, 12288, 3072, 16), (W8A8, 4608, 12288, 3072, 16),
          (W4A16, 1, 3072, 18432, 32), (W4A16, 16, 12288, 12288, 32), (W4A16, 16, 3072, 18432, 128), (W4A16, 70, 3072, 9216, 96)]


def test_the_lds_limit_is_raised_on_every_device(record):
    """A kernel that takes more than 64 KB of dynamic LDS needs the limit raised on the device it runs on: on the first
    device's word alone, a second GPU of the same process would have to launch without."""
    calls = [(dev, *s) for dev in (0, 1, 0, 5) for s in SHAPES]
    raised = {}
    big = set()
    for call, rec in zip(calls, record(calls)):
        assert any(r[0] == "launch" for r in rec), call
        for r in rec:
            if r[0] == "attr":
                raised[r[1], r[2]] = max(raised.get((r[1], r[2]), 0), r[3])
            else:
                assert r[1] == call[0]
                if r[6] > 65536:
                    big.add(r[2])
                    assert raised.get((r[1], r[2]), 0) >= r[6], (call, r)
    assert len(big) >= 8      # (the shapes do reach such kernels)


def test_w4a16_takes_sixteen_wavefronts_only_in_one_round(record):
    """A workgroup of sixteen wavefronts leaves no room for a second one on its CU, so a launch of more workgroups than CUs
    runs them one after the other where two of eight wavefronts would overlap."""
    #         M, K, N, rank, threads per workgroup: long K on one and two column blocks in one round, then beyond, then short K
    shapes = [(16, 12288, 3072, 32, 1024), (16, 12288, 12288, 32, 1024), (4, 6144, 12288, 16, 1024), (32, 6144, 8192, 32, 1024),
              (64, 8192, 8192, 32, 512), (40, 6144, 10240, 32, 512), (4, 6144, 30720, 32, 512), (4800, 6144, 32, 32, 512), (16, 3072, 12288, 32, 512)]
    for (M, K, N, r, threads), rec in zip(shapes, record([(0, W4A16, *s[:4]) for s in shapes])):
        launches = [x for x in rec if x[0] == "launch"]
        assert len(launches) == 1 and launches[0][5] == threads, (M, K, N, r, launches)
        assert threads == 512 or launches[0][3] * launches[0][4] <= 256, (M, K, N, r, launches)


OFFSETS = r"""
#include <stdio.h>
#include <initializer_list>
#include "layout.h"
using namespace svdq;
int main() {
    long checked = 0;
    // K-sharing kernels: every wavefront's loads up to the ring's depth past its last step; a block is a kilobyte
    for (int steps = 1; steps <= 40; ++steps)
        for (int KS : {4, 8, 16})
            for (int wave = 0; wave < KS; ++wave) {
                const int n = wave < steps ? (steps - wave + KS - 1) / KS : 0;
                for (int i = 0; i <= n + 6; ++i) {
                    const int st = kpar_step(wave, KS, i, n);
                    if (st < 0 || st >= steps || (i < n && st != wave + KS * i)) return printf("step %d of %d\n", st, steps), 1;
                    ++checked;
                }
            }
    // ring kernels: their tiles, the last tile of the padded rows and columns, every place of the ring, the last step
    const int tiles[5][2] = {{4, 8}, {6, 6}, {6, 4}, {4, 4}, {8, 8}};
    for (auto &t : tiles)
        for (int rows = 1; rows <= 9; ++rows)
            for (int cols = 1; cols <= 9; ++cols) {
                const int Mpad = rows * kRowPad, Npad = cols * kRowPad, steps = 3;
                for (int gm0 = 0; gm0 + t[0] * 32 <= Mpad; gm0 += t[0] * 32)
                    for (int gn0 = 0; gn0 + t[1] * 32 <= Npad; gn0 += t[1] * 32)
                        for (int j = 0; j < (t[0] + t[1] + 3) / 4 * 4; ++j) {
                            const long pad = j < t[0] ? Mpad : Npad, end = ring_offset(j, t[0], t[1], gm0, gn0) + (steps - 1) * pad * 32 + 1024;
                            if (end > steps * pad * 32) return printf("tile %d x %d place %d: %ld\n", t[0], t[1], j, end), 1;
                            ++checked;
                        }
            }
    // 128 x (32 blocks) tiles of the INT4 kernel: every tile of a launch (the last one of a row may reach past the padded columns), the last group.
    // A lane asks for nothing or for 16 bytes of its group's weight blocks, and what the tile has of them is asked for
    for (int blocks : {5, 6})
        for (int N = 16; N <= 12 * kRowPad; N += 16) {
            const int Npad = round_up(N, kRowPad), G = 3, pieces = mid_pieces(blocks);
            const long slab = (long)(Npad / 64) * kW4BBlock, whole = (long)w4_b_bytes(G, Npad);
            for (int gn0 = 0; gn0 < N; gn0 += 32 * blocks)
                for (int j = 7; j < (pieces + 3) / 4 * 4; ++j)
                    for (int lane = 0; lane < 64; ++lane) {
                        const MidPiece p = mid_piece(j, lane, pieces, 0, gn0, Npad);
                        const long want = gn0 / 64 * (long)kW4BBlock + (j - 7) * 1024 + lane * 16, first = p.base + (G - 1) * slab;
                        const bool asks = p.lane >= 0, wanted = j < pieces && want < slab;
                        if (p.base < 0 || first >= whole || (asks && first + p.lane + 16 > whole) || (!asks && p.lane != (int)0x80000000u) || asks != wanted || (asks && p.base + p.lane != want))
                            return printf("%d blocks, N %d, column %d, piece %d, lane %d: %ld of %ld\n", blocks, N, gn0, j, lane, first + p.lane, whole), 1;
                        ++checked;
                    }
        }
    for (int gm0 = 0; gm0 < 4 * kRowPad; gm0 += 128)
        for (int j = 0; j < 7; ++j)
            for (int lane = 0; lane < 64; ++lane)
                if (const MidPiece p = mid_piece(j, lane, mid_pieces(5), gm0, 0, kRowPad); p.base + p.lane != (long)w4_a_block(0, 4 * kRowPad, gm0) + j * 1024 + lane * 16 || p.base + p.lane + 16 > (long)w4_a_bytes(1, 4 * kRowPad))
                    return printf("row %d, piece %d\n", gm0, j), 1;
    return printf("ok %ld\n", checked), 0;
}
"""


def test_loads_that_ask_for_nothing_keep_their_offsets_inside_the_buffers(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "offsets.cpp", tmp_path / "offsets"
    src.write_text(OFFSETS)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(os.path.dirname(HERE), "paper_2411_05007_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


def _gemm_grid(rec):
    return [x for x in rec if x[0] == "launch"][-1][3]


@pytest.mark.parametrize("M,K,N,r,tiles", [(1800, 1152, 4608, 16, 15 * 18), (2048, 1536, 4608, 32, 16 * 18), (900, 320, 9216, 16, 8 * 36), (700, 320, 9216, 32, 6 * 36),
                                           (2048, 1600, 4608, 32, 32 * 72), (2048, 1536, 4608, 48, 32 * 72), (3000, 1536, 3072, 32, 47 * 48),      # more groups, a wider branch, square
                                           (2048, 384, 3072, 32, 16 * 48), (512, 320, 9216, 32, 8 * 144), (512, 320, 6144, 32, 4 * 96)])          # fewer tiles
def test_int4_few_groups_on_many_tiles_take_the_large_tiles(record, M, K, N, r, tiles):
    """The K-sharing kernel pays its fixed parts once per round of 512 workgroups, which few groups do not earn back: wide
    launches beyond four rounds up to 24 groups, any beyond two and a half up to five, take 128 x 256 tiles if the branch is
    narrow."""
    assert _gemm_grid(record([(0, INT4, M, K, N, r)])[0]) == tiles


@pytest.mark.parametrize("M,K,N,r,threads", [(900, 192, 4608, 64, 256), (256, 512, 12288, 16, 256), (2300, 320, 4608, 0, 256), (900, 576, 4608, 64, 1024), (16, 3072, 3072, 16, 1024)])
def test_w8a8_short_rows_take_the_walking_activation_kernel(record, M, K, N, r, threads):
    """The one-pass activation kernel deals a token's groups to sixteen wavefronts: at most eight groups leave half of them idle."""
    assert [x for x in record([(0, W8A8, M, K, N, r)])[0] if x[0] == "launch"][0][5] == threads


def _kernels(rec):
    return [x[2] for x in rec if x[0] == "launch"]


@pytest.mark.parametrize("fmt,M,K,N,r", [(FP4, 2, 4352, 240, 128), (FP4, 48, 4736, 160, 128), (FP4, 9, 4864, 160, 112), (INT4, 131, 5056, 5104, 112),
                                         (INT4, 72, 3008, 11840, 128), (INT4, 4, 12160, 144, 112), (STATIC, 119, 5184, 7712, 128)])
def test_runs_too_many_for_the_gemm_give_way_to_longer_ones(record, fmt, M, K, N, r):
    """The short runs of a small launch may leave more partial H than the workspace holds or than the tiles should read: then
    the longer runs, whose partial H the GEMM adds too, and not the meeting of a slice's runs in the activation kernel."""
    gemm = _kernels(record([(0, fmt, M, K, N, r)])[0])[-1]
    assert "kpar" in gemm and gemm.endswith(",true>"), gemm


@pytest.mark.parametrize("fmt,M,K,N,r,runs", [(FP4, 136, 640, 9248, 96, 1), (FP4, 713, 576, 1408, 32, 1), (INT4, 6, 576, 7136, 16, 1), (INT4, 365, 640, 6016, 96, 1),
                                              (INT4, 986, 704, 6544, 32, 1), (INT4, 217, 576, 2320, 32, 1), (FP4, 33, 640, 1040, 96, 2), (INT4, 33, 640, 1040, 96, 2), (INT4, 33, 832, 1040, 16, 2)])
def test_nine_to_twelve_groups_are_cut_for_small_tiles_only(record, fmt, M, K, N, r, runs):
    """Two runs' partial H are read by every tile: of a K this short only 32-row tiles (INT4: of a branch of 48 columns or more), and
    MXFP4's 64-row tiles, earn that back."""
    act = [x for x in record([(0, fmt, M, K, N, r)])[0] if x[0] == "launch"][0]
    assert act[2].startswith("act_kernel<") and act[3] == -(-M // 16) * runs, act


@pytest.mark.parametrize("M,K,N,r,runs", [(562, 3136, 9024, 64, False), (832, 3904, 5408, 64, False), (396, 9792, 11584, 64, False), (598, 4288, 9024, 32, False), (1810, 2112, 9584, 32, False),
                                          (452, 832, 8272, 64, True), (516, 832, 8912, 32, True), (512, 3072, 9216, 32, True)])
def test_wide_tiles_add_few_columns_of_partial_h(record, M, K, N, r, runs):
    gemm = _kernels(record([(0, INT4, M, K, N, r)])[0])[-1]
    assert gemm.startswith("gemm_w4a4_mid_kernel<") and gemm.endswith(",true>") == runs, gemm


@pytest.mark.parametrize("fmt,M,K,N,r,wide", [(FP4, 2595, 2560, 272, 128, False), (FP4, 2233, 3392, 512, 96, False), (STATIC, 3019, 7488, 304, 112, False), (STATIC, 4352, 11136, 416, 96, False),
                                              (INT4, 577, 2752, 2576, 128, False), (INT4, 2790, 2624, 400, 96, False), (INT4, 1905, 3648, 112, 96, False), (INT4, 622, 6144, 4576, 80, False),
                                              (FP4, 700, 2560, 2560, 128, True), (FP4, 1432, 9856, 2720, 128, True), (INT4, 4608, 12288, 3072, 128, True), (INT4, 1096, 9728, 1184, 128, True),
                                              (INT4, 1445, 5440, 416, 112, True), (INT4, 2419, 4160, 304, 96, True), (INT4, 1579, 5312, 448, 128, True), (INT4, 741, 12352, 2608, 80, True), (STATIC, 3875, 12352, 144, 128, True)])
def test_wide_branches_keep_their_kernel_off_launches_it_would_leave_cus_idle_in(record, fmt, M, K, N, r, wide):
    """Workgroups of 64 tokens with room for few runs' partial H are few, with long chains of groups: such launches take the
    kernel of 16-token workgroups."""
    assert _kernels(record([(0, fmt, M, K, N, r)])[0])[0].startswith("act_wide_kernel<") == wide


@pytest.mark.parametrize("M,K,N,r,walk", [(700, 4608, 1824, 48, True), (1464, 6080, 1520, 96, True), (700, 6208, 1824, 16, False), (1464, 4160, 1520, 16, True), (700, 4096, 1824, 48, False), (1464, 3072, 1520, 96, False)])
def test_int8_on_four_wavefronts_walks_a_long_k(record, M, K, N, r, walk):
    gemm = _kernels(record([(0, W8A8, M, K, N, r)])[0])[-1].split("<")[1].split(",")
    assert gemm[0] == "true" and gemm[3] == "4" and (gemm[5] == "true") == walk, gemm


@pytest.mark.parametrize("M,K,N,r,kernel", [(1719, 4928, 14448, 0, "gemm_w4a4_kernel<"), (3404, 5056, 7360, 16, "gemm_w4a4_kernel<"), (2191, 5056, 10816, 32, "gemm_w4a4_kernel<"),
                                            (4096, 4608, 1152, 32, "gemm_w4a4_mid_kernel<5,"), (2048, 3072, 3072, 32, "gemm_w4a4_mid_kernel<6,"), (1774, 9536, 10256, 16, "gemm_w4a4_mid_kernel<6,")])
def test_wide_tiles_take_four_rounds_at_most(record, M, K, N, r, kernel):
    assert _kernels(record([(0, INT4, M, K, N, r)])[0])[-1].startswith(kernel)


FORMATS = {"int4": INT4, "fp4": FP4, "w8a8": W8A8}
GPU_SHAPES = ([("int4", *s[:4], s[-1]) for s in G.TWO_SHARES] + [("w8a8", *s) for s in G.W8A8_LARGE + G.W8A8_LONG] + [("w8a8", *s[:4], k) for s in G.W8A8_SMALL for k in ("act_w8_small_kernel<", s[4])]
              + [("fp4", *s) for s in G.MXFP4_ROUNDS] + [(f, *s) for s in G.ONE_PASS for f in ("int4", "fp4")] + [("fp4", *s, "gemm_kpar_blocks_kernel<false,1,1,16,6,") for s in G.NARROW] + G.SPECIAL
              + [(f, *s, k) for f, s, k in G_CANARIES])


def test_the_gpu_tests_run_the_kernels_they_are_for(record):
    """A change of a rule must not turn a kernel's tests into tests of another kernel without a word."""
    calls = [(0, FORMATS[f], M, K, N, r) for f, M, K, N, r, _ in GPU_SHAPES]
    for call, rec in zip(GPU_SHAPES, record(calls)):
        assert any(k.startswith(call[-1]) for k in _kernels(rec)), (call, _kernels(rec))


def _wide_runs(rec, M):
    act = [x for x in rec if x[0] == "launch"][0]
    return act[3] // -(-M // 64) if act[2].startswith("act_wide_kernel<") else 0


def test_partial_h_lies_where_the_gpu_tests_of_wide_branches_expect_it(record):
    """Runs of the 64-token workgroups with an output of its own memory, at an odd address and in the input's: where the number does
    not change, the workspace holds them."""
    shapes = [(f, M, K, N, r, runs, other) for f, M, K, N, r, runs, other in G.WIDE] + [(f, M, K, K, r, runs, other) for f, M, K, r, runs, other in G.ANY_OUTPUT]
    recs = record([(0, FORMATS[f], M, K, N, r, 0, output) for f, M, K, N, r, *_ in shapes for output in (0, 1, 2)])
    for i, (f, M, K, N, r, runs, other) in enumerate(shapes):
        assert [_wide_runs(x, M) for x in recs[3 * i:3 * i + 3]] == [runs, other, other], shapes[i]


@pytest.mark.parametrize("M,K,N,r", [(512, 3072, 8192, 32), (1024, 3072, 4096, 32), (512, 3072, 9216, 32), (300, 3072, 2064, 48), (64, 12288, 12288, 16), (4608, 3072, 3072, 32)])
def test_the_static_workspace_runs_the_ordinary_launches(record, M, K, N, r):
    """Ordinary workspaces of small launches are larger than the static array for the room of a K split that such launches do
    not make: the static call does without that room, not without its launches."""
    mine, ordinary = record([(0, STATIC, M, K, N, r), (0, INT4, M, K, N, r)])
    assert [x[2:] for x in mine if x[0] == "launch"] == [x[2:] for x in ordinary if x[0] == "launch"]
