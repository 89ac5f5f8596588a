"""Which output tiles MXFP4 and INT8 launches take (csrc/layout.h, plan_gemm_fp4 and plan_kpar_blocks), and forwards that take them."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2411_05007_amd import svdq as S
from tests.test_gpu_parity import torch  # noqa: F401 (fixture)
from tests.test_gpu_small_launches import _block_format, _wide_branch
from tests.test_gpu_w8a8 import _random_layer, _run_and_compare
from tests.test_host_launches import FP4, HERE, INT4, W8A8, _gemm_grid, _kernels, record  # noqa: F401 (fixture)

FITS = r"""
#include <stdio.h>
#include <initializer_list>
#include "layout.h"
using namespace svdq;
int main() {
    const int rows[4] = {128, 192, 192, 128}, cols[4] = {256, 192, 128, 128};
    for (int M = 1; M <= 5000; M += M < 64 ? 1 : 37)
        for (int N = 16; N <= 13000; N += N < 640 ? 16 : 208)
            for (int G : {1, 18, 48, 192})
                for (int want : {0, 1, 3}) {
                    const GemmPlanFp4 p = plan_gemm_fp4(M, N, G, want);
                    const int tm = (M + rows[p.tile] - 1) / rows[p.tile], tn = (N + cols[p.tile] - 1) / cols[p.tile];
                    if (p.tiles != tm * tn || tm * rows[p.tile] > round_up(M, kRowPad) || tn * cols[p.tile] > round_up(N, kRowPad) || p.ksplit < 1 || (p.ksplit > 1 && p.tile != 0))
                        return printf("M %d, N %d, G %d, %d: tile %d, %d of them, split %d\n", M, N, G, want, p.tile, p.tiles, p.ksplit), 1;
                }
    return printf("ok\n"), 0;
}
"""


def test_tiles_fit_the_padded_rows_and_columns(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "fits.cpp", tmp_path / "fits"
    src.write_text(FITS)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(os.path.dirname(HERE), "paper_2411_05007_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout


@pytest.mark.parametrize("fmt,M,K,N,r,kernel,tiles", [
    (FP4, 4608, 3072, 9216, 32, "gemm_fp4_kernel<3,3,true>", 24 * 48), (W8A8, 3000, 3072, 9216, 16, "gemm_w8a8_kernel<3,3,true>", 16 * 48), (FP4, 4608, 3072, 3072, 32, "gemm_fp4_kernel<2,4,false>", 36 * 12),
    (FP4, 4406, 7168, 2304, 32, "gemm_fp4_kernel<3,2,false>", 23 * 18), (W8A8, 907, 5952, 7216, 16, "gemm_w8a8_kernel<3,3,true>", 5 * 38), (W8A8, 4608, 12288, 3072, 16, "gemm_w8a8_kernel<4,4,true>", 18 * 12),
    (FP4, 1024, 3072, 3072, 32, "gemm_fp4_kernel<2,2,false>", 8 * 24), (FP4, 1024, 4096, 3072, 32, "gemm_kpar_blocks_kernel<", 8 * 48), (FP4, 1024, 3072, 3072, 128, "gemm_kpar_blocks_kernel<", 8 * 48),
    (W8A8, 1558, 1152, 1952, 16, "gemm_w8a8_kernel<2,2,true>", 13 * 16), (W8A8, 1558, 1216, 1952, 16, "gemm_kpar_blocks_kernel<", 13 * 31)])
def test_which_tiles_a_launch_takes(record, fmt, M, K, N, r, kernel, tiles):  # noqa: F811
    rec = record([(0, fmt, M, K, N, r)])[0]
    assert _kernels(rec)[-1].startswith(kernel) and _gemm_grid(rec) == tiles, (_kernels(rec), _gemm_grid(rec))


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,K,N,r", [("fp4", 1141, 1984, 6928, 48), ("fp4", 641, 1088, 4240, 32), ("fp4", 299, 2368, 6160, 64), ("fp4", 257, 1024, 8208, 32), ("w8a8", 1900, 1984, 4528, 16), ("w8a8", 641, 1088, 4240, 32)])
def test_tiles_of_launches_that_took_others(torch, fmt, M, K, N, r):  # noqa: F811
    """Ragged last tiles of every shape, steps off the rounds of four, activations in one pass of eight tokens up to rank 64 and from 17 slices on."""
    if fmt == "fp4":
        return _wide_branch(torch, fmt, M, K, N, r)
    xb, w, ax, b = _random_layer(np.random.default_rng(7400 + M), M, K, N)
    _run_and_compare(torch, xb, S.svdq_w8a8_prepare(w, ax, r, bias=b), rows=np.r_[0:20, M - 140:M], what=f"w8a8 {M}x{K}x{N} r{r}")


@pytest.mark.parametrize("fmt,M,K,N,r,kpar", [
    (FP4, 16, 3072, 18432, 64, True), (FP4, 1, 3072, 32768, 32, True), (FP4, 129, 1024, 12800, 16, True), (FP4, 240, 1792, 8640, 32, True), (FP4, 96, 3072, 18432, 48, True), (FP4, 200, 1024, 12800, 64, True),
    (FP4, 241, 1792, 8640, 32, False), (FP4, 97, 3072, 18432, 48, False), (FP4, 200, 1152, 12800, 64, False), (FP4, 1, 1152, 25600, 0, False),
    (W8A8, 500, 1152, 6400, 0, True), (W8A8, 4, 1024, 16448, 32, True), (W8A8, 64, 1152, 18432, 32, True), (W8A8, 65, 1152, 18432, 32, False), (W8A8, 4, 1024, 16448, 16, False)])
def test_few_tokens_share_k(record, fmt, M, K, N, r, kpar):  # noqa: F811
    """257 to 512 tiles of 128 x 64: few tokens whose runs' partial H the K-sharing tiles add by themselves, and INT8 without a branch."""
    rec = record([(0, fmt, M, K, N, r)])[0]
    assert _kernels(rec)[-1].startswith("gemm_kpar_blocks_kernel<") == kpar, _kernels(rec)


@pytest.mark.parametrize("fmt,M,K,N,r,tile", [
    (W8A8, 4493, 1152, 19904, 16, "3,3"), (FP4, 2571, 1024, 25232, 32, "3,3"), (W8A8, 527, 640, 11136, 16, "2,2"), (W8A8, 2080, 1664, 2976, 16, "2,2"), (FP4, 3592, 1280, 1712, 32, "2,2"), (W8A8, 3728, 64, 34544, 16, "2,2"),
    (W8A8, 907, 5952, 7216, 16, "3,3"), (FP4, 892, 3456, 7232, 32, "3,3"), (FP4, 1800, 3072, 12288, 32, "3,3"), (W8A8, 2379, 320, 7008, 16, "3,3")])
def test_tiles_of_short_loops(record, fmt, M, K, N, r, tile):  # noqa: F811
    """192 x 192 tiles where a CU has several of them, 128 x 128 ones where it would have a single large one with a short loop, and for large INT8 launches of a few groups."""
    k = _kernels(record([(0, fmt, M, K, N, r)])[0])
    assert k[-1].startswith(("gemm_fp4_kernel<" if fmt == FP4 else "gemm_w8a8_kernel<") + tile + ","), k


# calls beside the lines that the tables of layout.h draw, with the activation kernel and the tiles that they take: ragged tokens, columns and groups
LINES = [("fp4", 17, 1088, 16464, 48, "act_kernel<", "gemm_kpar_blocks_kernel<"), ("fp4", 129, 1088, 8272, 32, "act_kernel<", "gemm_kpar_blocks_kernel<"), ("fp4", 97, 1216, 16464, 64, "act_tile_kernel<", "gemm_fp4_kernel<2,2,"),
         ("fp4", 301, 2112, 1040, 0, "act_kernel<", "gemm_kpar_blocks_kernel<"), ("fp4", 371, 2176, 528, 32, "act_kernel<", "gemm_kpar_blocks_kernel<"), ("fp4", 131, 1088, 23440, 16, "act_kernel<", "gemm_fp4_kernel<3,2,"),
         ("fp4", 257, 1088, 2064, 0, "act_onepass_kernel<", "gemm_kpar_blocks_kernel<"), ("int4", 1024, 2624, 1040, 32, "act_kernel<", "gemm_w4a4_kpar_kernel<"),
         ("w8a8", 33, 1088, 16464, 32, "act_w8_small_kernel<", "gemm_kpar_blocks_kernel<"), ("w8a8", 397, 1152, 5200, 0, "act_w8_small_kernel<", "gemm_kpar_blocks_kernel<"), ("w8a8", 201, 1088, 19984, 0, "act_w8_small_kernel<", "gemm_w8a8_kernel<2,2,"),
         ("w8a8", 201, 2624, 16528, 32, "act_w8_small_kernel<", "gemm_w8a8_kernel<"), ("w8a8", 2049, 192, 10768, 16, "act_kernel<", "gemm_w8a8_kernel<2,2,")]


@pytest.mark.parametrize("fmt,M,K,N,r,act,gemm", LINES)
def test_which_kernels_the_lines_choose(record, fmt, M, K, N, r, act, gemm):  # noqa: F811
    k = _kernels(record([(0, {"int4": INT4, "fp4": FP4, "w8a8": W8A8}[fmt], M, K, N, r)])[0])
    assert k[0].startswith(act) and k[-1].startswith(gemm), k


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,K,N,r", [s[:5] for s in LINES])
def test_forwards_beside_the_lines(torch, fmt, M, K, N, r):  # noqa: F811
    """Codes and scales exact, H and Y to the bounds of the formats' own tests."""
    if fmt == "int4":
        return _wide_branch(torch, fmt, M, K, N, r)
    _block_format(torch, fmt, M, K, N, r, None)


def test_int8_tiles_fit_the_padded_rows_and_columns(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "fits8.cpp", tmp_path / "fits8"
    src.write_text(FITS.replace("plan_gemm_fp4(M, N, G, want)", "plan_gemm_fp4(M, N, G, want, 32, true)").replace("{1, 18, 48, 192}", "{1, 7, 8, 18}"))
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(os.path.dirname(HERE), "paper_2411_05007_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok"), r.stdout
