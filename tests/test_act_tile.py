"""Activation kernel of 32-token workgroups (csrc/act_tile_kernel.hip): against the oracle at the sizes where its indexing can go wrong,
and on the CPU which calls take it."""
import numpy as np
import pytest

from oracle import svdq_oracle as O
from paper_2411_05007_amd import svdq as S
from tests.test_gpu_canaries import _check, _guarded
from tests.test_gpu_parity import torch  # noqa: F401 (fixture)
from tests.test_gpu_small_launches import _block_layer, _layer, _wide_branch
from tests.test_host_launches import FP4, INT4, STATIC, _kernels, record  # noqa: F401 (fixture)

# tokens off 32 (one and two in the last tile), groups off the four wavefronts and off the runs, last runs shorter than a round of the wavefronts,
# one, two and four blocks of 32 columns of H and ranks off them, partial H in the output's memory and in the workspace
EDGES = [("int4", 328, 1984, 7984, 112), ("int4", 431, 1024, 11664, 128), ("int4", 1337, 5376, 272, 48), ("int4", 2049, 2752, 416, 128), ("int4", 1501, 8256, 272, 16), ("int4", 1250, 4928, 512, 80),
         ("fp4", 1001, 3968, 432, 48), ("fp4", 97, 7040, 160, 128), ("fp4", 1337, 4032, 208, 64), ("fp4", 2049, 4288, 208, 112), ("fp4", 1025, 7360, 7184, 32)]


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,K,N,r", EDGES)
def test_tiles_of_32_tokens(torch, fmt, M, K, N, r):  # noqa: F811
    """Codes and scales exact, H and Y to the bounds of the other activation kernels' tests."""
    _wide_branch(torch, fmt, M, K, N, r)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt,M,K,N,r", [EDGES[0], EDGES[7]])
def test_tiles_of_32_tokens_stay_in_their_buffers_and_rows(torch, fmt, M, K, N, r):  # noqa: F811
    """Guarded output and workspace; a row with an infinity or a NaN becomes NaN, the others keep their bits."""
    rng = np.random.default_rng(6300 + M)
    layer = S.DeviceLayer(_layer(rng, K, N, r) if fmt == "int4" else _block_layer(rng, fmt, K, N, r))
    x = S.bf16_tensor_from_bits(O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)))
    n = layer.workspace(M).numel()
    big_ws, ws, big_y, y = _guarded(torch, layer, M, N, n)
    for _ in range(2):
        layer.forward(x, out=y, workspace=ws)
    _check(torch, big_ws, n, big_y, M, f"32 tokens {fmt}")
    want = y.clone()
    bad, rows = x.clone(), [0, 40, M - 1]
    for m, v in zip(rows, (float("inf"), float("nan"), float("-inf"))):
        bad[m, (7 * m + 3) % K] = v
    got = layer.forward(bad)
    rest = [m for m in range(M) if m not in rows]
    assert bool(torch.isnan(got[rows].float()).all())
    assert torch.equal(got[rest].view(torch.int16), want[rest].view(torch.int16))


@pytest.mark.gpu
def test_tiles_of_32_tokens_into_any_output(torch):  # noqa: F811
    """The output at an odd address and in the input's memory, where partial H goes elsewhere: sums in another order at most (perf/cases.py)."""
    M, K, r = 1500, 4096, 48
    rng = np.random.default_rng(6400)
    layer = S.DeviceLayer(_layer(rng, K, K, r))
    x = S.bf16_tensor_from_bits(O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)))
    y = layer.forward(x).float()
    odd = torch.empty(M * K + 8, dtype=torch.bfloat16, device=x.device)[1:1 + M * K].view(M, K)
    shared = x.clone()
    for src, out in ((x, odd), (shared, shared)):
        got = layer.forward(src, out=out).float()
        assert ((got - y).norm() / y.norm()).item() < 1.5e-4


def test_which_launches_take_tiles_of_32_tokens(record):  # noqa: F811
    """Cut runs whose partial H the GEMM does not add, unless there is room for too few of them: not where the 16-token workgroups fill the
    CUs with a short K, where 64-token ones are taken, or where one pass over K is enough."""
    fmts = {"int4": INT4, "fp4": FP4}
    took = [(0, fmts[f], *s) for f, *s in EDGES] + [(0, INT4, 512, 12288, 3072, 128), (0, STATIC, 905, 11136, 5264, 48)]
    other = [(0, INT4, 3246, 1408, 432, 64), (0, INT4, 4006, 2816, 2736, 64), (0, FP4, 2235, 1664, 768, 96), (0, FP4, 1500, 3072, 4608, 32), (0, INT4, 4608, 12288, 3072, 128), (0, INT4, 512, 3072, 3072, 64),
             (0, INT4, 512, 960, 9216, 128), (0, INT4, 328, 1984, 7984, 160), (0, INT4, 328, 1984, 7984, 112, 4 << 12), (0, INT4, 328, 1984, 7984, 112, 1)]
    recs = record(took + other)
    for c, rec in zip(took, recs):
        k = _kernels(rec)
        assert len(k) == 3 and k[0].startswith("act_tile_kernel<") and k[1] == "act_sum_h_kernel", (c, k)
    for c, rec in zip(other, recs[len(took):]):
        assert not any(k.startswith("act_tile") for k in _kernels(rec)), (c, _kernels(rec))


@pytest.mark.parametrize("fmt,M,K,N,r,tile", [("fp4", 128, 1024, 36864, 16, False), ("fp4", 171, 8192, 23408, 16, False), ("int4", 256, 1024, 36864, 16, False), ("int4", 64, 8192, 23408, 32, False),
                                              ("fp4", 400, 8192, 23408, 32, True), ("fp4", 16, 2048, 36864, 64, True), ("int4", 1, 4096, 36864, 128, True)])
def test_few_tokens_with_a_narrow_branch_keep_their_launches(record, fmt, M, K, N, r, tile):  # noqa: F811
    """Up to 256 tokens at ranks 16 and 32 the runs that meet in one launch are the faster ones."""
    k = _kernels(record([(0, {"int4": INT4, "fp4": FP4}[fmt], M, K, N, r)])[0])
    assert k[0].startswith("act_tile_kernel<") == tile, k
