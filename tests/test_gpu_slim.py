"""Up to 16 tokens with a workgroup for every 16 channels: rows of fewer stages than wavefronts and of several rounds of them, odd and even numbers of super-units, the
fewest and the most tokens and panels, a workgroup per compute unit and two on some; against a product in 64 bits.  Operands are small integers, so every
partial sum is exact."""
import pytest
import torch

from paper_2603_05232_amd import binding
from test_gpu_mid_tiles import _linear, _rows

pytestmark = pytest.mark.gpu

# tokens, channels, units per row, with a workspace
SHAPES = [(1, 5, 1, False), (16, 130, 2, False), (8, 300, 3, True), (9, 1000, 15, True), (15, 8 * 128, 16, True), (16, 32 * 128, 17, True), (7, 31 * 128 - 3, 33, True), (3, 22 * 128, 70, True),
          (1, 12 * 128 + 1, 111, True), (16, 640, 71, False), (5, 32 * 128 - 4, 130, False), (1, 33 * 128, 40, True), (6, 64 * 128 - 1, 15, True), (16, 40 * 128, 5, True)]
# beside them: longer split rows, more panels, more tokens, few panels of split rows
BESIDE = [(1, 12 * 128, 112, True), (16, 8 * 128, 57, True), (1, 33 * 128, 41, True), (16, 40 * 128, 7, True), (1, 65 * 128, 9, True), (17, 300, 16, True), (5, 7 * 128, 64, True)]


@pytest.mark.parametrize("dtype,N", [("i8", 4), ("bf16", 4), ("fp8", 3), ("fp16", 5)])
@pytest.mark.parametrize("M,O,units,with_ws", SHAPES + BESIDE)
def test_sixteen_channels(dtype, N, M, O, units, with_ws):
    for fused in ([True, False] if N == 4 else [False]):
        _linear(M, O, _rows(units, N, dtype, fused), N, dtype, fused, with_ws, units)


@pytest.mark.parametrize("dtype", ["i8", "fp16"])
@pytest.mark.parametrize("M,pad_x,pad_y", [(5, 16, 1), (16, 48, 4)])
def test_rows_with_gaps(dtype, M, pad_x, pad_y):
    """Token rows and rows of Y with other strides than their lengths; rows of an odd number of super-units, and non-finite weights behind them."""
    O, K = 6 * 128 - 5, 128 * 9 // (1 if dtype == "i8" else 2)
    td = torch.int8 if dtype == "i8" else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(pad_x)
    X = torch.randint(-3, 4, (M, K + pad_x), generator=gen, device="cuda").to(td)[:, :K]
    W = torch.where(torch.arange(K, device="cuda") % 8 < 6, torch.randint(-3, 4, (O, K), generator=gen, device="cuda"), 0)
    one = torch.ones(max(M, O), device="cuda") if dtype == "i8" else None
    wv, wm = binding.slide_decompose_fused(W.to(td), 4, dtype)
    wv = torch.cat([wv.view(torch.uint8).flatten(), torch.full((1 << 16,), 0x7F, dtype=torch.uint8, device="cuda")])
    out = torch.full((M, O + pad_y), 7.0, dtype=torch.bfloat16, device="cuda")
    binding.slide_sparse_gemm_fused(X, None if one is None else one[:M], wv, wm, None if one is None else one[:O], O, K, 4, dtype, out=out[:, :O])
    assert torch.equal(out[:, :O], (X.double() @ W.double().T).bfloat16())
    assert bool((out[:, O:] == 7.0).all())
