"""The 128-channel x 256-token tile kernel that lifts its tokens itself, at the edges of its pairs of super-units (odd and
even row lengths, fewer pairs than its rings hold to several rings) and of its tiles, on operand and result rows with
gaps, and as the rest behind whole rounds of 256 x 256 tiles; against a product in 64 bits.  Operands are small integers,
so every partial sum is exact in all types.  (More 128 x 128 tiles than compute units, at most one 128 x 256 tile for each.)"""
import pytest
import torch

from paper_2603_05232_amd import binding
from test_gpu_mid_tiles import _linear

pytestmark = pytest.mark.gpu


def _k(units, dtype):
    return 128 * units // (1 if dtype in ("i8", "fp8") else 2)


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("units", [1, 2, 3, 4, 5, 6, 7, 8, 9, 14])
def test_pairs_of_super_units(dtype, units):
    _linear(1100, 4224 - (units & 1) * 3, _k(units, dtype), 4, dtype, True, bool(units & 2), units)


EDGES = [(129, 129 * 128), (255, 140 * 128 - 1), (256, 256 * 128), (257, 86 * 128 + 8), (4097, 1000), (16300, 500)]


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("M,O", EDGES)
def test_edges_of_tiles(dtype, M, O):
    _linear(M, O, _k(5, dtype), 4, dtype, True, False, M)


# 8 token tiles: one round of 32 x 8 tiles of 256 x 256, the rest 25 panels x 8
REST = (2048, 32 * 256 + 3142)


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("units", [16, 17])
def test_rest_behind_whole_rounds(dtype, units):
    _linear(*REST, _k(units, dtype), 4, dtype, True, False, units)


@pytest.mark.parametrize("dtype", ["i8", "fp16"])
@pytest.mark.parametrize("pad_x,pad_y", [(16, 1), (128, 8), (48, 4)])
def test_rows_with_gaps(dtype, pad_x, pad_y):
    M, O, K = 700, 50 * 128 - 5, _k(3, dtype)
    td = torch.int8 if dtype == "i8" else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(pad_x)
    X = torch.randint(-3, 4, (M, K + pad_x), generator=gen, device="cuda").to(td)[:, :K]
    W = torch.where(torch.arange(K, device="cuda") % 8 < 6, torch.randint(-3, 4, (O, K), generator=gen, device="cuda"), 0)
    one = torch.ones(max(M, O), device="cuda") if dtype == "i8" else None
    wv, wm = binding.slide_decompose_fused(W.to(td), 4, dtype)
    out = torch.full((M, O + pad_y), 7.0, dtype=torch.bfloat16, device="cuda")
    binding.slide_sparse_gemm_fused(X, None if one is None else one[:M], wv, wm, None if one is None else one[:O], O, K, 4, dtype, out=out[:, :O])
    assert torch.equal(out[:, :O], (X.double() @ W.double().T).bfloat16())
    assert bool((out[:, O:] == 7.0).all())


# an infinite activation in the last super-unit, alone in its pair or not: the products that the row has, and no others
@pytest.mark.parametrize("dtype", ["bf16", "fp16"])
@pytest.mark.parametrize("units", [1, 3, 4, 5])
def test_infinity_in_the_last_super_unit(dtype, units):
    td = torch.bfloat16 if dtype == "bf16" else torch.float16
    M, O, K = 1100, 4224, 64 * units
    W = torch.where(torch.arange(K, device="cuda") % 8 < 6, 1.0, 0.0).to(td).expand(O, K).contiguous()
    X = torch.ones((M, K), dtype=td, device="cuda")
    X[5, K - 8 + 3] = float("inf")                          # a stored position: six of eight weights are kept
    wv, wm = binding.slide_decompose_fused(W, 4, dtype)
    Y = binding.slide_sparse_gemm_fused(X, None, wv, wm, None, O, K, 4, dtype)
    assert bool((Y[5] == float("inf")).all())
    Y[5] = K * 6 // 8
    assert bool((Y == K * 6 // 8).all())
