"""The GEMMs of launches with few output tiles, whose wavefronts share K (csrc/gemm_*kpar*): every variant that the
launch rule can pick, at the sizes where its indexing can go wrong - rows and columns off its tiles, a K of fewer groups
than wavefronts, group counts off the wavefront count, ranks with more steps than wavefronts - against the oracle, with
the bounds of the large kernel's tests (one bf16 rounding plus fp32 summation order)."""
import numpy as np
import pytest

from oracle import svdq_oracle as O
from paper_2411_05007_amd import svdq as S
from tests.test_gpu_parity import _run_and_compare, torch  # noqa: F401 (fixture)

pytestmark = pytest.mark.gpu


def _layer(rng, K, N, r):
    G = K // 64
    rinv = np.exp2(rng.uniform(-1, 1, K)).astype(np.float32)
    qw = rng.integers(-7, 8, size=(K, N)).astype(np.int8)
    sw = rng.uniform(5e-4, 4e-3, size=(G, N)).astype(np.float16)
    l1 = O.bf16_round((rng.standard_normal((K, r)) * 0.02).astype(np.float32))
    l2 = O.bf16_round((rng.standard_normal((r, N)) * 0.05).astype(np.float32))
    return S.svdq_pack(rinv, l1, l2, qw, sw, rng.standard_normal(N).astype(np.float32))


# rows per tile of the variant that the rule picks, and its tile count, follow each shape
@pytest.mark.parametrize("M,K,N,r,rows", [
    (1, 64, 16, 16, 32), (33, 128, 80, 16, 32), (31, 576, 1040, 144, 32), (64, 1088, 272, 0, 32),             # 32 rows, 8 wavefronts
    (290, 192, 2064, 32, 64), (257, 704, 3072, 144, 64), (320, 64, 2032, 16, 64),                             # 64 rows, 8 wavefronts
    (610, 192, 2064, 48, 64), (577, 832, 2320, 32, 64), (129, 64, 6160, 16, 64),                              # 64 rows, 4 wavefronts
    (45, 1600, 336, 112, 32), (17, 832, 80, 16, 32), (300, 6400, 1040, 64, 32),      # H added from two, three and five runs
    (520, 8256, 1984, 32, 128), (385, 8192, 3072, 160, 128),                                                  # 128 rows, 8 wavefronts
    (1000, 192, 3088, 80, 128), (897, 320, 3056, 16, 128), (1030, 64, 2736, 32, 128)])                        # 128 rows, 4 wavefronts
def test_every_variant_at_its_edges(torch, M, K, N, r, rows):  # noqa: F811
    rng = np.random.default_rng(5200 + M + K + N)
    prep = _layer(rng, K, N, min(r, K // 16 * 16, N))
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, rng.choice(K, max(1, K // 100), replace=False)] *= 50
    plan = S.svdq_debug_launch_plan(M, prep.shape)
    assert (plan["gemm_tiles"], plan["gemm_ksplit"]) == (-(-M // rows) * -(-N // 64), 1)
    print(f"small launch: M={M} K={K} N={N} r={prep.shape.rank}, {rows}-row tiles", flush=True)
    sample = np.unique(np.concatenate([np.arange(min(M, 40)), np.arange(max(0, M - 40), M), rng.integers(0, M, 60)]))
    _run_and_compare(torch, O.bf16_round(x), prep, rows=sample, what=f"small {M}x{K}x{N}", window=False)


# 128 x 160 and 128 x 192 tiles whose two shares of wavefronts take the even and the odd groups (csrc/gemm_w4a4_mid_kernel.hip): odd
# and even counts of either share's groups, rank steps that the shares divide unevenly, H ready-made and added from runs, columns
# past the padded ones, ragged M and N
TWO_SHARES = [(454, 448, 8272, 48, 160, "gemm_w4a4_mid_kernel<5,false>"), (579, 576, 6576, 32, 160, "gemm_w4a4_mid_kernel<5,false>"), (452, 832, 8272, 64, 160, "gemm_w4a4_mid_kernel<5,true>"),
              (457, 512, 8336, 0, 160, "gemm_w4a4_mid_kernel<5,false>"), (514, 448, 8976, 48, 192, "gemm_w4a4_mid_kernel<6,false>"), (516, 832, 8912, 32, 192, "gemm_w4a4_mid_kernel<6,true>"),
              (577, 640, 8176, 16, 192, "gemm_w4a4_mid_kernel<6,false>")]


@pytest.mark.parametrize("M,K,N,r,cols", [s[:5] for s in TWO_SHARES])
def test_two_shares_of_a_wide_tile(torch, M, K, N, r, cols):  # noqa: F811
    rng = np.random.default_rng(5700 + M + K + N)
    prep = _layer(rng, K, N, r)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, rng.choice(K, max(1, K // 100), replace=False)] *= 50
    plan = S.svdq_debug_launch_plan(M, prep.shape)
    assert (plan["gemm_tiles"], plan["gemm_ksplit"]) == (-(-M // 128) * -(-N // cols), 1)
    print(f"wide tile: M={M} K={K} N={N} r={r}, {cols} columns", flush=True)
    sample = np.unique(np.concatenate([np.arange(40), np.arange(M - 70, M), rng.integers(0, M, 60)]))
    _run_and_compare(torch, O.bf16_round(x), prep, rows=sample, what=f"wide {M}x{K}x{N}", window=False)


@pytest.mark.parametrize("M,K,N,r", [(5, 64, 16, 16), (6, 64, 48, 48), (17, 576, 1008, 64), (33, 1088, 9232, 32), (4, 704, 18448, 48),     # one, two, three column blocks
                                     (2, 6208, 80, 80), (19, 6144, 1040, 32), (3, 6208, 272, 0),                                        # sixteen wavefronts
                                     (5, 6208, 8240, 32), (9, 6208, 8240, 16),                                                         # sixteen wavefronts, two column blocks
                                     (4500, 6208, 32, 32),                                                                             # the same K in more than one round: eight
                                     (16, 320, 400, 256), (70, 256, 144, 96),                                                            # H from a launch of its own
                                     (2, 32768, 16, 16), (7, 32768, 32, 32)])                                                            # 1 / lambda fills the LDS
def test_w4a16_at_its_edges(torch, M, K, N, r):  # noqa: F811
    """Rows off the five and sixteen of a pass, column tails, fewer groups than wavefronts, every launch variant; bound:
    one bf16 rounding plus the fp32 summation of K products (test_gpu_w4a16.py)."""
    from tests.test_gpu_w4a16 import _run
    rng = np.random.default_rng(5300 + M + K + N)
    r = min(r, N // 16 * 16, K // 16 * 16)
    print(f"w4a16 edges: M={M} K={K} N={N} r={r}", flush=True)
    _run(torch, O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)), _layer(rng, K, N, r), f"w4a16 {M}x{K}x{N} r{r}")


# (the rule of the two block formats; the last column: rows per tile for MXFP4 and for INT8)
@pytest.mark.parametrize("M,K,N,r,rows", [
    (1, 64, 16, 16, (32, 32)), (33, 128, 80, 16, (32, 32)), (31, 576, 1040, 144, (32, 32)), (64, 1088, 272, 0, (32, 32)),
    (290, 192, 2064, 32, (64, 64)), (257, 704, 3072, 144, (64, 64)), (320, 64, 2032, 16, (64, 64)),
    (610, 192, 2064, 48, (128, 64)), (577, 832, 2320, 32, (128, 64)), (129, 64, 6160, 16, (128, 64)),
    (33, 3136, 80, 16, (32, 32)), (20, 6080, 144, 32, (32, 32)), (50, 2048, 272, 64, (32, 32)),      # groups off the wavefronts that hold K in registers
    (70, 2112, 208, 48, (32, 32)), (40, 2432, 144, 128, (32, 32)), (300, 3136, 2064, 32, (64, 64)),      # H added from runs
    (520, 8256, 1984, 32, (128, 128)), (1000, 192, 3088, 80, (128, 128)), (897, 320, 3056, 16, (128, 128))])
@pytest.mark.parametrize("fmt", ["fp4", "w8a8"])
def test_block_formats_at_their_edges(torch, fmt, M, K, N, r, rows):  # noqa: F811
    """Bounds: those of test_gpu_fp4.py and test_gpu_w8a8.py (exact codes and scales, one bf16 rounding plus fp32 summation order)."""
    _block_format(torch, fmt, M, K, N, r, (rows[0], 64))


# tiles of the launches that fill the chip: 192 x 128, 128 x 128 (K off four steps, fewer steps than the ring has stages, ragged M and N)
@pytest.mark.parametrize("M,K,N,r,tile", [(1337, 192, 9040, 32, (192, 128)), (1300, 64, 9232, 0, (192, 128)), (1000, 320, 9040, 48, (128, 128)), (970, 64, 9104, 16, (128, 128))])
@pytest.mark.parametrize("fmt", ["fp4", "w8a8"])
def test_block_formats_on_smaller_tiles(torch, fmt, M, K, N, r, tile):  # noqa: F811
    _block_format(torch, fmt, M, K, N, r, tile)


# one activation workgroup per 16 tokens with K in its wavefronts' registers (64 to 256 slices): fewer groups than
# wavefronts, group counts off sixteen in every variant, no projection, the last slice of a launch ragged
# (the first shape: INT4 only; MXFP4's small tiles add the walking kernel's runs)
ONE_PASS = [(1009, 704, 272, 16, "act_"), (1009, 704, 9232, 16, "act_onepass_kernel<"), (1009, 1088, 9232, 32, "act_onepass_kernel<"), (1500, 3136, 9232, 16, "act_onepass_kernel<"),
            (2050, 6080, 272, 32, "act_onepass_kernel<"), (4095, 128, 144, 0, "act_onepass_kernel<")]


@pytest.mark.parametrize("M,K,N,r", [s[:4] for s in ONE_PASS])
@pytest.mark.parametrize("fmt", ["int4", "fp4"])
def test_activation_in_one_pass(torch, fmt, M, K, N, r):  # noqa: F811
    if fmt == "fp4":
        return _block_format(torch, fmt, M, K, N, r, None)
    rng = np.random.default_rng(5500 + M + K + N)
    prep = _layer(rng, K, N, r)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, rng.choice(K, max(1, K // 100), replace=False)] *= 50
    sample = np.unique(np.concatenate([np.arange(40), np.arange(M - 40, M), rng.integers(0, M, 60)]))
    print(f"one pass: M={M} K={K} N={N} r={r}", flush=True)
    _run_and_compare(torch, O.bf16_round(x), prep, rows=sample, what=f"one pass {M}x{K}x{N}", window=False)


# INT8 on 256 x 256 tiles (csrc/w8a8_kernels.hip): last rows and columns of a tile, steps off the ring, the shortest K, all 256 CUs, three ranks
W8A8_LARGE = [(2561, 4672, 5136, 48, "gemm_w8a8_kernel<4,4,true>"), (3841, 4608, 3856, 16, "gemm_w8a8_kernel<4,4,true>"), (2310, 4864, 6160, 0, "gemm_w8a8_kernel<4,4,true>")]


@pytest.mark.parametrize("M,K,N,r", [s[:4] for s in W8A8_LARGE])
def test_w8a8_on_large_tiles(torch, M, K, N, r):  # noqa: F811
    _block_format(torch, "w8a8", M, K, N, r, None)


# wide branches, 64 tokens to an activation workgroup (csrc/act_wide_kernel.hip): tokens off 64, groups off the runs, last runs of one and two
# groups (fewer than the ring has stages), ranks off 128; the runs' partial H in the output's memory or in the workspace.  The last number: how
# many runs there are where the output cannot hold them
WIDE = [("int4", 2001, 2752, 4672, 112, 8, 0), ("int4", 1500, 2816, 6160, 80, 8, 0), ("int4", 1001, 5632, 3088, 128, 15, 15), ("int4", 1500, 5632, 528, 80, 15, 15), ("int4", 3010, 4672, 272, 128, 10, 10),
        ("fp4", 577, 2752, 2576, 112, 8, 7), ("fp4", 1001, 4672, 4672, 80, 13, 0), ("fp4", 2001, 4672, 528, 128, 13, 13), ("fp4", 577, 2624, 4112, 112, 7, 7), ("fp4", 3010, 4672, 272, 128, 8, 8)]


@pytest.mark.parametrize("fmt,M,K,N,r", [s[:5] for s in WIDE])
def test_wide_branches_in_64_token_workgroups(torch, fmt, M, K, N, r):  # noqa: F811
    _wide_branch(torch, fmt, M, K, N, r)


# the same ranks in 16-token workgroups, whose partial H the GEMM adds
@pytest.mark.parametrize("M,K,N,r", [(577, 2560, 1040, 128), (1100, 2624, 528, 80), (700, 5632, 144, 112), (3010, 4672, 272, 128)])
@pytest.mark.parametrize("fmt", ["int4", "fp4"])
def test_wide_branches(torch, fmt, M, K, N, r):  # noqa: F811
    _wide_branch(torch, fmt, M, K, N, r)


def _wide_branch(torch, fmt, M, K, N, r):  # noqa: F811
    if fmt == "fp4":
        return _block_format(torch, fmt, M, K, N, r, None)
    rng = np.random.default_rng(5800 + M + K + N)
    prep = _layer(rng, K, N, r)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, rng.choice(K, max(1, K // 100), replace=False)] *= 50
    sample = np.unique(np.concatenate([np.arange(40), np.arange(M - 70, M), rng.integers(0, M, 60)]))
    print(f"wide branch: M={M} K={K} N={N} r={r}", flush=True)
    _run_and_compare(torch, O.bf16_round(x), prep, rows=sample, what=f"wide branch {M}x{K}x{N}", window=False)


# square layers, so that the output can be the input; runs in the output's memory, and where it cannot hold them (in the workspace, or none:
# another kernel).  The third takes that other kernel anyhow
ANY_OUTPUT = [("int4", 2001, 4672, 128, 13, 0), ("fp4", 700, 2560, 128, 7, 5), ("int4", 640, 2560, 128, 0, 0)]


@pytest.mark.parametrize("fmt,M,K,r", [s[:4] for s in ANY_OUTPUT])
def test_wide_branch_into_any_output(torch, fmt, M, K, r):  # noqa: F811
    """The output's memory holds partial sums only where it can: not where it is the input's, and not at an odd address.  Bound:
    sums in another order, 2e-5 in the 2-norm (see perf/cases.py)."""
    rng = np.random.default_rng(5900)
    layer = S.DeviceLayer(_block_layer(rng, fmt, K, K, r) if fmt == "fp4" else _layer(rng, K, K, r))
    x = S.bf16_tensor_from_bits(O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)))
    y = layer.forward(x).float()
    odd = torch.empty(M * K + 8, dtype=torch.bfloat16, device=x.device)[1:1 + M * K].view(M, K)
    for out in (odd, x.clone()):
        got = layer.forward(x if out is odd else out, out=out).float()
        assert ((got - y).norm() / y.norm()).item() < 1.5e-4


# one shape for every kernel that adds up runs, shares K or stages its operands: the kernel it is for follows
SPECIAL = [("int4", 1500, 5632, 528, 80, "act_wide_kernel<0>"), ("fp4", 577, 2752, 2576, 112, "act_wide_kernel<1>"), ("int4", 452, 832, 8272, 64, "gemm_w4a4_mid_kernel<5,true>"),
           ("int4", 579, 576, 6576, 32, "gemm_w4a4_mid_kernel<5,false>"), ("w8a8", 290, 3136, 2064, 32, "act_w8_small_kernel<2,2>"), ("w8a8", 67, 4160, 1552, 32, "gemm_kpar_blocks_kernel<true,1,1,16,6,false,true>"),
           ("fp4", 33, 3520, 1552, 128, "gemm_kpar_blocks_kernel<false,1,1,16,6,false,true>"), ("w8a8", 2561, 4672, 5136, 48, "gemm_w8a8_kernel<4,4,true>")]


@pytest.mark.parametrize("fmt,M,K,N,r", [s[:5] for s in SPECIAL])
def test_infinities_and_nan_stay_in_their_rows(torch, fmt, M, K, N, r):  # noqa: F811
    """A row of X with an infinity or a NaN gives a row of NaN (its H is infinite or NaN, and infinity less its own bf16 part is
    NaN); every other row is what it is without them, bit for bit."""
    rng = np.random.default_rng(5950 + M + K + N)
    layer = S.DeviceLayer(_layer(rng, K, N, r) if fmt == "int4" else _block_layer(rng, fmt, K, N, r))
    x = S.bf16_tensor_from_bits(O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)))
    print(f"infinities and NaN: {fmt} M={M} K={K} N={N} r={r}", flush=True)
    want = layer.forward(x).clone()
    rows = sorted({0, 5, M // 2, M - 2, M - 1})
    bad = x.clone()
    for i, m in enumerate(rows):
        bad[m, int(rng.integers(0, K))] = (float("inf"), float("nan"), float("-inf"))[i % 3]
    got = layer.forward(bad)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(want.float()).all())
    assert bool(torch.isnan(got[rows].float()).all())
    rest = [m for m in range(M) if m not in rows]
    assert torch.equal(got[rest].view(torch.int16), want[rest].view(torch.int16))


# INT8: four tokens to a quantizing workgroup beside workgroups that project runs of K (csrc/act_w8_small_kernel.hip): tokens off four and
# sixteen, half a unit of 128 channels at the end, every number of units per wavefront, one and two rank steps and none, a GEMM that adds
# the runs on every kind of its tiles (32 x 32 ones among them) and one that needs H whole
W8A8_SMALL = [(1, 1472, 528, 16, "gemm_kpar_blocks_kernel<true,1,2,8,6,false,true>"), (5, 1408, 1040, 32, "gemm_kpar_blocks_kernel<true,1,1,16,6,false,true>"),
              (18, 2112, 4176, 0, "gemm_kpar_blocks_kernel<true,1,1,16,6,false,false>"), (67, 4160, 1552, 32, "gemm_kpar_blocks_kernel<true,1,1,16,6,false,true>"),
              (130, 6208, 2064, 16, "gemm_kpar_blocks_kernel<true,1,2,8,6,false,true>"), (3, 12288, 784, 32, "gemm_kpar_blocks_kernel<true,1,2,8,6,false,true>"),
              (290, 3136, 2064, 32, "gemm_kpar_blocks_kernel<true,2,2,8,4,false,true>"), (600, 640, 1552, 16, "gemm_kpar_blocks_kernel<true,2,2,8,4,false,true>"),
              (700, 3136, 1840, 16, "gemm_kpar_blocks_kernel<true,2,2,4,4,false,true>"), (1030, 1216, 2064, 32, "gemm_kpar_blocks_kernel<true,4,2,4,2,false,true>"),
              (520, 8256, 3056, 32, "gemm_kpar_blocks_kernel<true,4,2,8,2,false,true>"), (700, 576, 6160, 32, "act_sum_h_kernel"), (1100, 3200, 4112, 16, "act_sum_h_kernel")]


@pytest.mark.parametrize("M,K,N,r", [s[:4] for s in W8A8_SMALL])
def test_w8a8_small_batches(torch, M, K, N, r):  # noqa: F811
    _block_format(torch, "w8a8", M, K, N, r, None)


# INT8, four wavefronts that share a long K: steps off the wavefronts and the sets requested ahead, 64- and 128-row tiles, H ready-made and from runs
W8A8_LONG = [(690, 4160, 1840, 48, "gemm_kpar_blocks_kernel<true,2,2,4,4,true,false>"), (700, 6208, 1808, 16, "gemm_kpar_blocks_kernel<true,2,2,4,4,false,true>"),
             (1450, 4224, 1520, 96, "gemm_kpar_blocks_kernel<true,4,2,4,2,true,false>"), (1463, 4352, 1488, 32, "gemm_kpar_blocks_kernel<true,4,2,4,2,true,true>")]


@pytest.mark.parametrize("M,K,N,r", [s[:4] for s in W8A8_LONG])
def test_w8a8_long_k_on_four_wavefronts(torch, M, K, N, r):  # noqa: F811
    _block_format(torch, "w8a8", M, K, N, r, None)


# MXFP4 on 32 x 32 tiles with sixteen wavefronts: K off four steps, fewer steps than the wavefronts ask ahead, ragged M and N, ranks with
# more steps than a wavefront has, H ready-made and added from runs
NARROW = [(1, 3328, 1040, 32), (33, 3520, 1552, 128), (64, 6144, 2064, 0), (17, 8256, 4112, 48)]


@pytest.mark.parametrize("M,K,N,r", NARROW)
def test_mxfp4_on_narrow_tiles(torch, M, K, N, r):  # noqa: F811
    _block_format(torch, "fp4", M, K, N, r, (32, 32))


def _block_layer(rng, fmt, K, N, r):
    rinv = np.exp2(rng.uniform(-1, 1, K)).astype(np.float32)
    l1 = O.bf16_round((rng.standard_normal((K, r)) * 0.02).astype(np.float32))
    l2 = O.bf16_round((rng.standard_normal((r, N)) * 0.05).astype(np.float32))
    bias = rng.standard_normal(N).astype(np.float32)
    if fmt == "fp4":
        return S.svdq_fp4_pack(rinv, l1, l2, rng.integers(0, 16, size=(K, N)).astype(np.uint8), rng.integers(110, 118, size=(K // 32, N)).astype(np.uint8), bias)
    return S.svdq_w8a8_pack(rinv, l1, l2, rng.integers(-127, 128, size=(K, N)).astype(np.int8), rng.uniform(5e-5, 4e-4, N).astype(np.float16), bias)


def _block_format(torch, fmt, M, K, N, r, tile):  # noqa: F811
    from tests import test_gpu_fp4, test_gpu_w8a8
    rng = np.random.default_rng(5400 + M + K + N)
    r = min(r, K // 16 * 16, N)
    rinv = np.exp2(rng.uniform(-1, 1, K)).astype(np.float32)
    l1 = O.bf16_round((rng.standard_normal((K, r)) * 0.02).astype(np.float32))
    l2 = O.bf16_round((rng.standard_normal((r, N)) * 0.05).astype(np.float32))
    bias = rng.standard_normal(N).astype(np.float32)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, rng.choice(K, max(1, K // 100), replace=False)] *= 50
    sample = np.unique(np.concatenate([np.arange(min(M, 40)), np.arange(max(0, M - 40), M), rng.integers(0, M, 60)]))
    print(f"block formats: {fmt} M={M} K={K} N={N} r={r}", flush=True)
    if fmt == "fp4":
        prep = S.svdq_fp4_pack(rinv, l1, l2, rng.integers(0, 16, size=(K, N)).astype(np.uint8), rng.integers(110, 118, size=(K // 32, N)).astype(np.uint8), bias)
        plan = S.svdq_debug_launch_plan(M, prep.shape)
        assert tile is None or (plan["gemm_tiles"], plan["gemm_ksplit"]) == (-(-M // tile[0]) * -(-N // tile[1]), 1)
        test_gpu_fp4._run_and_compare(torch, O.bf16_round(x), prep, rows=sample, what=f"fp4 small {M}x{K}x{N}")
    else:
        prep = S.svdq_w8a8_pack(rinv, l1, l2, rng.integers(-127, 128, size=(K, N)).astype(np.int8), rng.uniform(5e-5, 4e-4, N).astype(np.float16), bias)
        test_gpu_w8a8._run_and_compare(torch, O.bf16_round(x), prep, rows=sample, what=f"w8a8 small {M}x{K}x{N}")


@pytest.mark.parametrize("M,K,N,rows", [(64, 1088, 272, 32), (290, 704, 2064, 64), (577, 832, 2320, 64), (520, 8256, 1984, 128), (897, 320, 3056, 128)])
def test_int4_group_sums_are_exact(torch, M, K, N, rows):  # noqa: F811
    """Every integer group sum of the K-sharing INT4 kernel, bit for bit, through its output: column n has the scale 1 in
    group n % G and 0 in the others, a token's scale is 1 (its largest value is 7), and twelve non-zero channels per
    token and group keep a sum within 49 + 11 * 14 = 203, a whole number that bf16 holds."""
    G = K // 64
    rng = np.random.default_rng(5600 + M)
    x = np.zeros((M, G, 64), np.int64)
    at = np.argsort(rng.random((M, G, 64)), axis=2)[:, :, :12]
    v = rng.integers(-2, 3, size=(M, G, 12))
    v[:, :, 0] = rng.choice([-7, 7], (M, G))
    np.put_along_axis(x, at, v, axis=2)
    qw = rng.integers(-7, 8, size=(K, N)).astype(np.int8)
    sw = (np.arange(G)[:, None] == np.arange(N)[None, :] % G).astype(np.float16)
    prep = S.svdq_pack(np.ones(K, np.float32), np.zeros((K, 0), np.uint16), np.zeros((0, N), np.uint16), qw, sw, np.zeros(N, np.float32))
    plan = S.svdq_debug_launch_plan(M, prep.shape)
    assert (plan["gemm_tiles"], plan["gemm_ksplit"]) == (-(-M // rows) * -(-N // 64), 1)
    print(f"group sums: M={M} K={K} N={N}, {rows}-row tiles", flush=True)
    layer = S.DeviceLayer(prep)
    y = layer.forward(S.bf16_tensor_from_bits(O.bf16_round(x.reshape(M, K).astype(np.float32))))
    torch.cuda.synchronize()
    want = np.empty((M, N), np.int64)
    for g in range(G):
        want[:, g::G] = x[:, g] @ qw.reshape(G, 64, N)[g][:, g::G].astype(np.int64)
    assert np.abs(want).max() > 100
    assert np.array_equal(O.bf16_to_f32(S.bits_from_bf16_tensor(y)), want.astype(np.float32))


# MXFP4 in large tiles of every shape: K loops of one, two and three steps more than whole rounds of four, of fewer than four, a rank that
# is no power of two; launches whose wavefronts share K: steps off the rounds of two, four and six
MXFP4_ROUNDS = [(1530, 320, 12272, 32, "gemm_fp4_kernel<3,3,true>"), (1530, 704, 12272, 48, "gemm_fp4_kernel<3,3,true>"), (4100, 192, 3088, 16, "gemm_fp4_kernel<2,4,false>"),
                (1337, 1472, 9200, 32, "gemm_fp4_kernel<3,2,false>"), (2040, 1728, 3072, 0, "gemm_fp4_kernel<2,2,false>"), (1000, 2240, 5136, 32, "gemm_fp4_kernel<2,2,false>"),
                (257, 1984, 2064, 32, "gemm_kpar_blocks_kernel<false,2,2,4,4,false,true>"), (100, 2368, 3088, 64, "gemm_kpar_blocks_kernel<false,1,2,8,6,false,true>"),
                (1024, 1856, 3072, 16, "gemm_kpar_blocks_kernel<false,4,2,4,2,false,true>")]


@pytest.mark.parametrize("M,K,N,r", [s[:4] for s in MXFP4_ROUNDS])
def test_mxfp4_steps_off_the_rounds(torch, M, K, N, r):  # noqa: F811
    _block_format(torch, "fp4", M, K, N, r, None)
