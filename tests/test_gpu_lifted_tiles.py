"""The 256 x 256 tile kernel over lifted rows at the edges of its ring (rows of few units, and the shortest that go elsewhere), of
its tiles and of its rounds, against a product in 64 bits.  Operands are small integers, so every partial sum is exact in
all types."""
import pytest
import torch

from paper_2603_05232_amd import binding
from test_gpu_mid_tiles import _linear

pytestmark = pytest.mark.gpu


def _k(units, N, dtype):
    """A row length whose lifted row is `units` units of 128 bytes long, the last block cut short."""
    es = 1 if dtype in ("i8", "fp8") else 2
    blocks = max(1, 128 * units // es // (4 * (N - 1)))
    return blocks * 2 * N - 1


# 17 x 9 tiles: one partial round; the last tiles hold 52 tokens and 121 to 128 channels
@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("units", [1, 2, 3, 4, 5, 6, 7, 8, 11])
def test_units(dtype, units):
    _linear(2100, 4224 - units, _k(units, 3 + units % 4, dtype), 3 + units % 4, dtype, False, False, units)


# more tiles than compute units (256): tiles that follow one another in a workgroup, with tokens and channels that end
# inside a tile, rows of fewer units than the ring holds among them.  32 x 36 tiles: four rounds and a half; 2 x 256 and 17 x 15
# tiles: two rounds and one, the channels behind them go to other tiles.
ROUNDS = [(8100, 9000, 1), (8100, 9000, 2), (8100, 9000, 3), (8100, 9000, 4), (8100, 9000, 5), (8100, 9000, 7), (257, 66000, 6)]
ONE_ROUND_AND_REST = [(4300, 4400, 3), (4300, 4400, 4), (4300, 4400, 5)]


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16"])
@pytest.mark.parametrize("M,O,units", ROUNDS + ONE_ROUND_AND_REST)
def test_rounds(dtype, M, O, units):
    _linear(M, O, _k(units, 4, dtype), 4, dtype, False, False, units)


# an infinite activation in the last block, in rows that are completed with zeros (one to three units of 64 lifted elements) and in longer
# ones: the products that the row has, and no others
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("blocks,units", [(5, 1), (10, 2), (16, 3), (21, 4), (37, 7)])
def test_infinity_in_the_last_block(dtype, blocks, units):
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    M, O, K = 2100, 4224, 8 * blocks
    W = torch.where(torch.arange(K, device="cuda") % 8 < 6, 1.0, 0.0).to(td).expand(O, K).contiguous()
    X = torch.ones((M, K), dtype=torch.bfloat16, device="cuda")
    X[5, K - 8 + 3] = float("inf")                          # a stored position: six of eight weights are kept
    XL, _ = binding.act_lift_quant(X, 4, dtype)
    assert XL.shape[1] == 64 * units
    wv, wm = binding.slide_decompose(W, 4, dtype)
    Y = binding.slide_sparse_gemm(XL, None, wv, wm, None, O, dtype)
    assert bool((Y[5] == float("inf")).all())
    Y[5] = K * 6 // 8
    assert bool((Y == K * 6 // 8).all())
