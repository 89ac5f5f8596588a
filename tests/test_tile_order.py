"""The order in which workgroups take the output tiles (csrc/layout.h, gemm_tile_of), with tile counts that 8 does not divide."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import svdq_oracle as O
from tests.test_gpu_parity import _run_and_compare, torch  # noqa: F401 (fixture)
from tests.test_gpu_small_launches import _block_format, _layer
from tests.test_host_launches import FP4, HERE, INT4, W8A8, _gemm_grid, _kernels, record  # noqa: F401 (fixture)

WALK = r"""
#include <stdio.h>
#include <vector>
#include "layout.h"
int main() {
    for (int from : {0, 40, 1000})
        for (int tm = 1; tm <= 27; ++tm)
            for (int tn = 1; tn <= 27; ++tn) {
                std::vector<int> seen(tm * tn, 0);
                std::vector<int> last(8, -1);
                for (int b = 0; b < tm * tn; ++b) {
                    int m, n;
                    svdq::gemm_tile_of(b, tm, tn, from, m, n);
                    if (m < 0 || m >= tm || n < 0 || n >= tn || seen[m * tn + n]++) return printf("%d x %d, from %d: workgroup %d takes %d, %d\n", tm, tn, from, b, m, n), 1;
                    // an XCD's tiles follow one another: band by band of eight rows, column by column
                    const int rows = tm - m / 8 * 8 < 8 ? tm - m / 8 * 8 : 8, id = m / 8 * 8 * tn + n * rows + m % 8;
                    if ((tm * tn % 8 == 0 || tm * tn >= from) && last[b % 8] >= 0 && id != last[b % 8] + 1) return printf("%d x %d: workgroup %d leaves its run\n", tm, tn, b), 1;
                    last[b % 8] = id;
                }
            }
    return printf("ok\n"), 0;
}
"""


def test_every_tile_is_taken_once_and_an_xcd_owns_a_run(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(os.path.dirname(HERE), "paper_2411_05007_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


FROM = r"""
#include <stdio.h>
#include <initializer_list>
#include "layout.h"
int main() {
    for (int i8 = 0; i8 < 2; ++i8)
        for (int G : {1, 16, 17, 24, 25, 192})
            for (int N : {16, 4096, 4112, 36864}) {
                const int tn = (N + 127) / 128;
                const bool few = N <= 4096 && G <= (i8 ? 16 : 24);
                for (int tm : {3, 11, 101}) {
                    const int total = tm * tn;
                    int m, n;
                    svdq::gemm_tile_of(1, tm, tn, svdq::xcd_order_from(i8, G, N), m, n);      // (the second tile of the first band, or the first one of the second XCD's run)
                    if (total > 16 && total % 8 && (m == 1 && n == 0) != (few && total < 600)) return printf("i8 %d, G %d, %d x %d: the second workgroup takes %d, %d\n", i8, G, tm, tn, m, n), 1;
                }
            }
    return printf("ok\n"), 0;
}
"""


def test_few_columns_of_short_rows_stay_in_launch_order(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "from.cpp", tmp_path / "from"
    src.write_text(FROM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", os.path.join(os.path.dirname(HERE), "paper_2411_05007_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout


# tiles past a multiple of eight: INT4 in one round and persistent, above the line and below it, then the two block formats
REST = [(INT4, 4400, 128, 4400, 16, 512), (INT4, 2732, 256, 9232, 64, 814), (INT4, 1635, 384, 7088, 16, 364), (FP4, 2900, 192, 4400, 16, 414), (W8A8, 2900, 192, 4400, 16, 414)]


def test_their_launches(record):  # noqa: F811
    for (fmt, M, K, N, r, tiles), rec in zip(REST, record([(0, *s[:5]) for s in REST])):
        print(fmt, M, K, N, r, _kernels(rec)[-1], _gemm_grid(rec))
        assert _gemm_grid(rec) == tiles, (_kernels(rec), _gemm_grid(rec))


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,K,N,r", [s[:5] for s in REST])
def test_every_tile_is_written(torch, fmt, M, K, N, r):  # noqa: F811
    if fmt != INT4:
        return _block_format(torch, {FP4: "fp4", W8A8: "w8a8"}[fmt], M, K, N, r, None)
    rng = np.random.default_rng(6700 + M)
    rows = np.unique(np.concatenate([np.arange(0, M, 61), np.arange(M - 8, M)]))
    print(f"tile order: M={M} K={K} N={N} r={r}", flush=True)
    _run_and_compare(torch, O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)), _layer(rng, K, N, r), rows=rows, window=False, what=f"tile order {M}x{K}x{N}")
