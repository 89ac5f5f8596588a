"""Forwards that run as one launch (csrc/fused_small_kernel.hip): against the oracle at the sizes where its indexing can go wrong, and on
the CPU which calls take it."""
import numpy as np
import pytest

from oracle import svdq_oracle as O
from paper_2411_05007_amd import svdq as S
from tests.test_gpu_canaries import _check, _guarded
from tests.test_gpu_parity import torch  # noqa: F401 (fixture)
from tests.test_gpu_small_launches import _block_format, _block_layer, _layer
from tests.test_host_launches import FP4, INT4, STATIC, W8A8, _kernels, record  # noqa: F401 (fixture)

# tokens off the tile's 32 and the load's 8; groups off the eight wavefronts and the two requested ahead; columns off 64, one column of
# tiles that stores every group's codes, more columns of tiles than groups, no 16-bit branch, half an operand of it
EDGES = [(1, 1024, 16, 16), (33, 1088, 80, 32), (31, 1152, 1040, 0), (256, 1152, 1152, 32), (9, 1472, 2064, 16), (70, 1728, 272, 32), (40, 1792, 64, 32), (17, 1280, 8208, 32)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,r", EDGES)
@pytest.mark.parametrize("fmt", ["int4", "fp4"])
def test_one_launch_at_its_edges(torch, fmt, M, K, N, r):  # noqa: F811
    """Codes and scales exact, H and Y to the bounds of the two-launch forward (one bf16 rounding plus fp32 summation order)."""
    print(f"one launch: {fmt} M={M} K={K} N={N} r={r}", flush=True)
    if fmt == "fp4":
        return _block_format(torch, fmt, M, K, N, r, None)
    from tests.test_gpu_parity import _run_and_compare
    rng = np.random.default_rng(6100 + M + K + N)
    x = rng.standard_normal((M, K)).astype(np.float32)
    x[:, rng.choice(K, K // 100, replace=False)] *= 50
    x[M // 2, 64:128] = 0.0
    _run_and_compare(torch, O.bf16_round(x), _layer(rng, K, N, r), what=f"one launch {M}x{K}x{N}", window=True)


@pytest.mark.gpu
@pytest.mark.parametrize("fmt", ["int4", "fp4"])
def test_one_launch_stays_in_its_buffers_and_rows(torch, fmt):  # noqa: F811
    """Guarded output and workspace; a row with an infinity or a NaN becomes NaN, the others keep their bits; an output in the input's
    memory (two launches) differs by summation order only, 2e-6 to 3.5e-5 in the 2-norm: held to 1.5e-4, the tolerance of perf/cases.py."""
    M, K, N, r = 70, 1152, 1152, 32
    rng = np.random.default_rng(6200)
    layer = S.DeviceLayer(_layer(rng, K, N, r) if fmt == "int4" else _block_layer(rng, fmt, K, N, r))
    x = S.bf16_tensor_from_bits(O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)))
    n = layer.workspace(M).numel()
    big_ws, ws, big_y, y = _guarded(torch, layer, M, N, n)
    for _ in range(2):
        layer.forward(x, out=y, workspace=ws)
    _check(torch, big_ws, n, big_y, M, f"one launch {fmt}")
    want = y.clone()
    bad, rows = x.clone(), [0, 40, 69]
    for m, v in zip(rows, (float("inf"), float("nan"), float("-inf"))):
        bad[m, 7 * m + 3] = v
    got = layer.forward(bad)
    rest = [m for m in range(M) if m not in rows]
    assert bool(torch.isnan(got[rows].float()).all())
    assert torch.equal(got[rest].view(torch.int16), want[rest].view(torch.int16))
    inplace = x.clone()
    layer.forward(inplace, out=inplace)
    assert ((inplace.float() - want.float()).norm() / want.float().norm()).item() < 1.5e-4


def test_which_forwards_run_as_one_launch(record):  # noqa: F811
    """Small batches with a K of 16 to 28 groups and a branch of at most 32 columns, unless the output shares memory with the input or
    an option asks for a part of the two launches."""
    one = [(fmt, *s) for fmt in (INT4, STATIC, FP4) for s in EDGES]
    other = [(INT4, 32, 960, 1152, 32), (FP4, 32, 1856, 1152, 32), (INT4, 32, 1152, 1152, 48), (INT4, 300, 1152, 2064, 32), (FP4, 2048, 1152, 1152, 32), (W8A8, 32, 1152, 1152, 16),
             (INT4, 32, 1152, 1152, 32, 1), (INT4, 32, 1152, 1152, 32, 2), (FP4, 32, 1152, 1152, 32, 1 << 8), (INT4, 32, 1152, 1152, 32, 4 << 12), (INT4, 32, 1152, 1152, 32, 0, 2), (FP4, 32, 1152, 1152, 32, 0, 2)]
    recs = record([(0, *c) for c in one + other])
    for c, rec in zip(one, recs):
        assert [k.split("<")[0] for k in _kernels(rec)] == ["fused_small_kernel"], (c, _kernels(rec))
    for c, rec in zip(other, recs[len(one):]):
        assert len(_kernels(rec)) >= 2 and not any(k.startswith("fused") for k in _kernels(rec)), (c, _kernels(rec))
    odd = record([(0, INT4, 32, 1152, 1152, 32, 0, 1)])[0]      # an output at an odd address is stored to as by the other kernels
    assert len(_kernels(odd)) == 1
