"""The 256 x 256 tile kernel that lifts its tokens itself, at the edges of its pairs of super-units (odd and even row
lengths, one pair to several), of its tiles and of its rounds, against a product in 64 bits.  Operands are small integers, so
every partial sum is exact in all types."""
import pytest
import torch

from paper_2603_05232_amd import binding
from test_gpu_mid_tiles import _linear

pytestmark = pytest.mark.gpu


# 17 x 9 tiles: one partial round; the last tiles hold 52 tokens and 124 or 127 channels
@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("units", [1, 2, 3, 4, 5, 6, 7, 9])
def test_pairs_of_super_units(dtype, units):
    _linear(2100, 4224 - (units & 1) * 3, 128 * units // (1 if dtype in ("i8", "fp8") else 2), 4, dtype, True, False, units)


# more tiles than compute units (256): tiles that follow one another in a workgroup, with tokens and channels that end
# inside a tile, and rows of one pair, where every load of the next tile is requested by the first pair of the one before.
# 32 x 36 tiles: four rounds and a half; 2 x 256 and 17 x 15 tiles: two rounds and one, the channels behind them go to other tiles.
ROUNDS = [(8100, 9000, 1), (8100, 9000, 2), (8100, 9000, 3), (8100, 9000, 4), (8100, 9000, 5), (257, 66000, 5), (257, 66000, 6)]
ONE_ROUND_AND_REST = [(4300, 4400, 1), (4300, 4400, 2), (4300, 4400, 3)]


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16"])
@pytest.mark.parametrize("M,O,units", ROUNDS + ONE_ROUND_AND_REST)
def test_rounds(dtype, M, O, units):
    _linear(M, O, 128 * units // (1 if dtype in ("i8", "fp8") else 2), 4, dtype, True, False, units)


# an infinite activation in the last super-unit, alone in its pair or not: the products that the row has, and no others
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("units", [3, 4])
def test_infinity_in_the_last_super_unit(dtype, units):
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    M, O, K = 2100, 4224, 64 * units
    W = torch.where(torch.arange(K, device="cuda") % 8 < 6, 1.0, 0.0).to(td).expand(O, K).contiguous()
    X = torch.ones((M, K), dtype=td, device="cuda")
    X[5, K - 8 + 3] = float("inf")                          # a stored position: six of eight weights are kept
    wv, wm = binding.slide_decompose_fused(W, 4, dtype)
    Y = binding.slide_sparse_gemm_fused(X, None, wv, wm, None, O, K, 4, dtype)
    assert bool((Y[5] == float("inf")).all())
    Y[5] = K * 6 // 8
    assert bool((Y == K * 6 // 8).all())
