"""Small unsplit tiles (one or two fragments of a panel x 32 to 128 tokens): each tile at the edges of its tokens, channels and rings, rows that do not divide into its groups of wavefronts, with and
without a workspace; against a product in 64 bits.  Operands are small integers, so every partial sum is exact."""
import pytest
import torch

from paper_2603_05232_amd import binding
from test_gpu_mid_tiles import _linear, _rows

pytestmark = pytest.mark.gpu

# tokens, channels, units per row, with a workspace, fragments, blocks of 32 tokens
SHAPES = [(8, 36 * 128, 30, True, 1, 1), (16, 64 * 128 - 1, 40, True, 1, 1), (17, 5, 4, True, 1, 1), (32, 64 * 128, 5, False, 1, 1), (33, 32 * 128 - 3, 6, True, 1, 1), (64, 28 * 128, 28, True, 1, 1), (100, 300, 19, True, 1, 1), (1000, 2 * 128 - 5, 9, True, 1, 1), (63, 1000, 131, False, 1, 1),
          (12, 96 * 128 - 2, 12, True, 2, 1), (20, 65 * 128, 7, True, 2, 1), (64, 64 * 128 - 1, 30, True, 2, 1), (129, 24 * 128 + 4, 22, True, 2, 1), (31, 127 * 128, 90, False, 2, 1), (700, 5 * 128, 4, False, 2, 1),
          (49, 65 * 128, 3, True, 2, 2), (65, 60 * 128 - 7, 3, True, 2, 2), (250, 32 * 128, 41, True, 2, 2), (128, 64 * 128 - 9, 100, False, 2, 2),
          (256, 42 * 128, 35, True, 2, 3), (193, 42 * 128 - 5, 8, False, 2, 3), (90, 127 * 128, 2, True, 2, 3),
          (128, 128 * 128 - 100, 12, True, 2, 4), (512, 32 * 128, 31, True, 2, 4), (97, 120 * 128, 5, False, 2, 4), (4000, 4 * 128 - 3, 6, True, 2, 4)]
# beside them: split rows of more lines, fewer units than groups and three with up to 48 tokens, more panels, and few tokens
BESIDE = [(33, 65 * 128, 3, True), (48, 727, 3, False), (32, 20 * 128, 60, True), (40, 300, 64, True), (128, 20 * 128, 64, True), (40, 300, 1, True), (64, 129 * 128, 5, False), (129, 65 * 128, 20, False), (16, 300, 90, True), (16, 65 * 128, 11, True)]


@pytest.mark.parametrize("dtype,N", [("i8", 4), ("bf16", 4), ("fp8", 3), ("fp16", 5)])
@pytest.mark.parametrize("M,O,units,with_ws", [s[:4] for s in SHAPES] + BESIDE)
def test_tiles(dtype, N, M, O, units, with_ws):
    for fused in ([True, False] if N == 4 else [False]):
        _linear(M, O, _rows(units, N, dtype, fused), N, dtype, fused, with_ws, units)


@pytest.mark.parametrize("dtype", ["i8", "fp16"])
@pytest.mark.parametrize("M,O,pad_x,pad_y", [(40, 6 * 128 - 5, 16, 1), (150, 20 * 128 - 5, 48, 4), (256, 42 * 128 - 2, 128, 3), (300, 40 * 128 - 5, 32, 8)])
def test_rows_with_gaps(dtype, M, O, pad_x, pad_y):
    K = 128 * 9 // (1 if dtype == "i8" else 2)
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
