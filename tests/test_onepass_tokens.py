"""One-pass activation kernel with workgroups of eight tokens (csrc/act_onepass_kernel.hip): against the oracles at the sizes where its
indexing can go wrong, the same bits as with sixteen, and on the CPU which calls take it."""
import numpy as np
import pytest

from oracle import svdq_oracle as O
from paper_2411_05007_amd import svdq as S
from tests.test_gpu_canaries import _check, _guarded
from tests.test_gpu_parity import torch  # noqa: F401 (fixture)
from tests.test_gpu_small_launches import _block_layer, _layer, _wide_branch
from tests.test_gpu_w8a8 import _random_layer, _run_and_compare
from tests.test_host_launches import FP4, INT4, W8A8, record  # noqa: F401 (fixture)


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,r", [(1337, 3072, 3088, 16), (2041, 640, 2320, 32), (2000, 3072, 2320, 32), (801, 2112, 9216, 64), (797, 1088, 9216, 0), (1009, 1024, 9216, 48)])
def test_int8_eight_tokens(torch, M, K, N, r):  # noqa: F811
    """Tokens off 8 and off 16, groups off the sixteen wavefronts, two, three and six groups per wavefront, one, two and four column blocks of H and none."""
    rng = np.random.default_rng(7100 + M)
    xb, w, ax, b = _random_layer(rng, M, K, N)
    rows = np.r_[0:24, M // 2, M - 20:M]
    _run_and_compare(torch, xb, S.svdq_w8a8_prepare(w, ax, r, bias=b), rows=rows, what=f"w8a8 {M}x{K}x{N} r{r}")


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,K,N,r", [("int4", 1009, 1088, 9232, 32), ("int4", 2041, 6080, 272, 16), ("int4", 1672, 2048, 9232, 32), ("fp4", 1017, 1984, 9232, 16), ("fp4", 2041, 6080, 2576, 32)])
def test_blocks_eight_tokens(torch, fmt, M, K, N, r):  # noqa: F811
    _wide_branch(torch, fmt, M, K, N, r)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,K,N,r", [("w8a8", 1337, 3072, 3088, 16), ("int4", 1009, 1088, 9232, 32), ("fp4", 1017, 1984, 9232, 16)])
def test_eight_tokens_are_those_of_a_larger_batch(torch, fmt, M, K, N, r):  # noqa: F811
    """A token's codes, scales and H do not depend on the tokens beside it: the first M rows of a batch whose workgroups have sixteen.  Guarded buffers;
    rows with an infinity or a NaN leave the others' bits as they are."""
    rng = np.random.default_rng(7200 + M)
    if fmt == "w8a8":
        _, w, ax, b = _random_layer(rng, 8, K, N)
        layer = S.DeviceLayer(S.svdq_w8a8_prepare(w, ax, r, bias=b))
    else:
        layer = S.DeviceLayer(_layer(rng, K, N, r) if fmt == "int4" else _block_layer(rng, fmt, K, N, r))
    large = S.bf16_tensor_from_bits(O.bf16_round(rng.standard_normal((2064, K)).astype(np.float32)))
    layer.forward(large)
    want = [np.asarray(t)[:M].copy() for t in layer.debug_act()]
    x = large[:M].clone()
    n = layer.workspace(M).numel()
    big_ws, ws, big_y, y = _guarded(torch, layer, M, N, n)
    for _ in range(2):
        layer.forward(x, out=y, workspace=ws)
    _check(torch, big_ws, n, big_y, M, f"eight tokens {fmt}")
    layer.forward(x)
    for a, t in zip(layer.debug_act(), want):
        a = np.ascontiguousarray(a)
        assert np.array_equal(a.view(np.uint8), np.ascontiguousarray(t).view(np.uint8))
    bad, rows = x.clone(), [0, 13, M - 1]
    for m, v in zip(rows, (float("inf"), float("nan"), float("-inf"))):
        bad[m, (7 * m + 3) % K] = v
    got, rest = layer.forward(bad), [m for m in range(M) if m not in rows]
    assert torch.equal(got[rest].view(torch.int16), layer.forward(x)[rest].view(torch.int16))


def test_which_launches_take_eight_tokens(record):  # noqa: F811
    """While they are one round of the CUs."""
    eight = [(0, W8A8, 1337, 3072, 9216, 16), (0, W8A8, 2000, 3072, 3072, 16), (0, INT4, 1009, 1088, 9232, 32), (0, FP4, 2048, 3072, 3072, 32)]
    sixteen = [(0, W8A8, 2049, 3072, 9216, 16), (0, W8A8, 4608, 3072, 9216, 32), (0, INT4, 2050, 6080, 272, 32), (0, FP4, 4096, 3072, 3072, 32)]
    for c, rec in zip(eight + sixteen, record(eight + sixteen)):
        grids = [(r[2], int(r[3])) for r in rec if r[0] == "launch" and r[2].startswith("act_onepass_kernel<")]
        tok = 8 if c in eight else 16
        assert len(grids) == 1 and grids[0][0].endswith(f",{tok}>") and grids[0][1] == -(-c[2] // tok), (c, grids)


# launches whose tiles could add partial H: group counts off sixteen and off the rounds of the loops, ragged last workgroups and tiles
INSTEAD = [("int4", 371, 1088, 2064, 32), ("int4", 777, 1984, 4624, 16), ("int4", 1029, 3008, 3088, 32), ("int4", 2041, 2112, 3088, 32), ("fp4", 371, 1088, 3088, 32), ("fp4", 1029, 3008, 1552, 32)]


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,K,N,r", INSTEAD)
def test_one_pass_instead_of_partial_h(torch, fmt, M, K, N, r):  # noqa: F811
    _wide_branch(torch, fmt, M, K, N, r)


def test_which_launches_leave_no_partial_h(record):  # noqa: F811
    fmts = {"int4": INT4, "fp4": FP4}
    for c, rec in zip(INSTEAD, record([(0, fmts[f], *s) for f, *s in INSTEAD])):
        k = [r[2] for r in rec if r[0] == "launch"]
        assert len(k) == 2 and k[0].startswith("act_onepass_kernel<") and k[0].endswith(",8>"), (c, k)
    other = [(0, INT4, 512, 3072, 3072, 32), (0, INT4, 368, 1152, 2064, 32), (0, INT4, 1024, 3136, 3072, 32), (0, INT4, 1024, 1152, 2064, 48), (0, FP4, 512, 1856, 3072, 16), (0, INT4, 1024, 1152, 2064, 32, 4 << 12)]
    for c, rec in zip(other, record(other)):
        assert not any(r[2].startswith("act_onepass") for r in rec if r[0] == "launch"), (c, rec)


@pytest.mark.parametrize("M,K,N,one_pass", [(667, 3008, 64, False), (300, 2240, 2800, False), (500, 3072, 6400, False), (1008, 2048, 1536, False), (1009, 2048, 1536, True), (300, 1536, 3072, True), (300, 1600, 3072, False)])
def test_mxfp4_without_a_branch(record, M, K, N, one_pass):  # noqa: F811
    """Nothing has to meet over K, so cut runs cost no second launch: one pass of rows up to K = 1536, and where workgroups of sixteen tokens would fill a quarter of the CUs."""
    k = [r[2] for r in record([(0, FP4, M, K, N, 0)])[0] if r[0] == "launch"]
    assert k[0].startswith("act_onepass_kernel<") == one_pass, k


@pytest.mark.parametrize("fmt,M,K,N,r,one_pass", [
    (FP4, 371, 2560, 2560, 32, False), (FP4, 512, 2112, 2048, 32, False), (FP4, 1024, 3072, 1024, 32, False), (FP4, 771, 3072, 64, 32, False), (INT4, 1024, 3072, 1536, 32, False),
    (FP4, 371, 2560, 3072, 32, True), (FP4, 771, 2560, 1536, 32, True), (FP4, 1025, 3072, 1024, 32, True), (FP4, 371, 2048, 64, 32, True), (INT4, 1025, 3072, 1536, 32, True), (INT4, 1024, 2560, 1536, 32, True), (INT4, 1024, 3072, 4608, 32, True), (INT4, 512, 2048, 512, 16, True)])
def test_partial_h_stays_where_few_tiles_read_it(record, fmt, M, K, N, r, one_pass):  # noqa: F811
    """Three groups to a wavefront: tiles of 32 or 64 rows (MXFP4), and up to 1024 tokens, which the runs' workgroups take in one round."""
    k = [r[2] for r in record([(0, fmt, M, K, N, r)])[0] if r[0] == "launch"]
    assert len(k) == 2 and k[0].startswith("act_onepass_kernel<") == one_pass, k


@pytest.mark.parametrize("M,K,N,r,one_pass", [(16, 2048, 39936, 0, False), (512, 1536, 9984, 0, False), (768, 3072, 9984, 0, False), (4, 3072, 33024, 32, False), (256, 2624, 19968, 32, False),
                                              (4, 3072, 33024, 16, True), (257, 3072, 19968, 32, True), (4, 2560, 33024, 32, True), (769, 3072, 9984, 0, True)])
def test_int8_launches_that_quantize_beside_the_projection(record, M, K, N, r, one_pass):  # noqa: F811
    """Large tiles: without a branch there is no sum to make; few tokens of a K above 2560 with more than 16 columns of H."""
    k = [x[2] for x in record([(0, W8A8, M, K, N, r)])[0] if x[0] == "launch"]
    assert k[-1].startswith("gemm_w8a8_kernel<") and k[0].startswith("act_onepass_kernel<" if one_pass else "act_w8_small_kernel<"), k
