"""W4A16 with the parts of X^ in LDS (csrc/w4a16_kernel.hip, PARTS): one to five rows, and the sizes up to which they fit."""
import numpy as np
import pytest

from oracle import svdq_oracle as O
from paper_2411_05007_amd import svdq as S
from tests.test_gpu_parity import torch  # noqa: F401 (fixture)
from tests.test_gpu_small_launches import _layer
from tests.test_host_launches import W4A16, _kernels, record  # noqa: F401 (fixture)

# fewer channels than threads, several turns of the workgroup and a last one that is not full, passes of five rows and a rest, H's shares behind the parts and in
# their place, no H, H from a launch of its own
EDGES = [(1, 64, 16, 16), (2, 192, 80, 32), (5, 1088, 1040, 48), (7, 1600, 272, 32), (1, 16448, 48, 16), (2, 6144, 336, 48), (5, 3904, 144, 64), (3, 6720, 80, 0), (4, 2112, 9232, 32), (3, 2048, 208, 128)]


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,r", EDGES)
def test_parts_at_their_edges(torch, M, K, N, r):  # noqa: F811
    """Bound: one bf16 rounding plus the fp32 summation of K products (test_gpu_w4a16.py)."""
    from tests.test_gpu_w4a16 import _run
    rng = np.random.default_rng(6500 + M + K + N)
    print(f"w4a16 parts: M={M} K={K} N={N} r={r}", flush=True)
    _run(torch, O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)), _layer(rng, K, N, min(r, N, K)), f"w4a16 {M}x{K}x{N} r{r}")


@pytest.mark.gpu
def test_infinities_keep_to_their_rows_and_products(torch):  # noqa: F811
    """An infinite input gives its row the signed infinities of the codes it meets, as the sums of products do, and no other row anything."""
    M, K, N = 4, 1088, 272
    rng = np.random.default_rng(6600)
    prep = _layer(rng, K, N, 0)
    layer = S.DeviceLayer(prep)
    x = S.bf16_tensor_from_bits(O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)))
    want = layer.forward_w4a16(x).clone()
    bad = x.clone()
    bad[2, 700] = float("inf")
    got = layer.forward_w4a16(bad)
    q = S.svdq_unpack(prep)["qw"][700].astype(np.float32)
    assert torch.equal(got[[0, 1, 3]].view(torch.int16), want[[0, 1, 3]].view(torch.int16))
    row = got[2].float().cpu().numpy()
    assert np.all(np.isposinf(row[q > 0])) and np.all(np.isneginf(row[q < 0])) and np.all(np.isnan(row[q == 0]))


def test_which_calls_keep_the_parts_in_lds(record):  # noqa: F811
    calls = [(*s, True) for s in EDGES if s[0] <= 5] + [(5, 4160, 1040, 32, False), (2, 12288, 272, 16, False), (6, 1088, 272, 32, False), (16, 3072, 18432, 32, False)]
    for (M, K, N, r, parts), rec in zip(calls, record([(0, W4A16, M, K, N, r) for M, K, N, r, _ in calls])):
        assert _kernels(rec)[-1].endswith(",true>") == parts, (M, K, N, r, _kernels(rec))


def test_where_parts_in_lds_would_cost(record):  # noqa: F811
    """More workgroups than CUs, two of which share a CU only without the parts; loops of one group per wavefront and few rows."""
    calls = [(5, 2048, 36864, 32, False), (4, 2560, 24592, 16, False), (3, 3072, 27648, 32, False), (5, 3072, 36864, 0, False), (3, 4096, 36864, 32, False), (5, 4096, 30720, 0, False),
             (3, 2048, 36864, 32, True), (2, 3072, 36864, 16, True), (4, 3072, 30720, 0, True), (4, 4096, 24592, 32, True), (2, 6144, 30720, 32, True), (5, 3072, 24576, 32, True),
             (5, 2048, 27648, 64, True), (3, 3072, 36864, 48, True), (2, 3072, 17408, 64, True),
             (1, 512, 36864, 16, False), (2, 448, 9216, 32, False), (3, 320, 18432, 0, False), (1, 128, 272, 16, False), (1, 512, 80, 64, False), (2, 512, 9216, 48, False),
             (1, 576, 36864, 16, True), (2, 512, 9216, 32, True), (3, 384, 18432, 64, True), (4, 64, 18432, 32, True), (1, 512, 128, 32, True)]
    for (M, K, N, r, parts), rec in zip(calls, record([(0, W4A16, M, K, N, r) for M, K, N, r, _ in calls])):
        assert _kernels(rec)[-1].endswith(",true>") == parts, (M, K, N, r, _kernels(rec))


@pytest.mark.gpu
@pytest.mark.parametrize("M,K,N,r", [(5, 2048, 24656, 16), (4, 2112, 24592, 0), (1, 128, 272, 16), (2, 448, 1040, 48), (3, 64, 144, 64)])
def test_parts_in_the_loop_where_lds_would_cost(torch, M, K, N, r):  # noqa: F811
    """Bound: as for the parts in LDS."""
    from tests.test_gpu_w4a16 import _run
    rng = np.random.default_rng(6700 + M + K + N)
    print(f"w4a16 parts in the loop: M={M} K={K} N={N} r={r}", flush=True)
    _run(torch, O.bf16_round(rng.standard_normal((M, K)).astype(np.float32)), _layer(rng, K, N, min(r, N, K)), f"w4a16 {M}x{K}x{N} r{r}")
