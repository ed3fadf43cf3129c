"""Few tokens as a stream of weights: workgroups of five, six and eight fragments on layers of more panels than compute units (256 compute
units: 257 to 320, 321 to 384 and 385 to 512 panels), token tiles of 32, 64 and 128, and of four fragments on fewer panels, with and without split
rows; against a product in 64 bits.  Operands are small integers, so every partial sum is exact."""
import pytest
import torch

from paper_2603_05232_amd import binding
from test_gpu_mid_tiles import _linear, _rows

pytestmark = pytest.mark.gpu

# tokens, channels, units per row, fused
SHAPES = [(1, 257 * 128 - 5, 16, True), (9, 320 * 128, 17, False), (32, 321 * 128 - 3, 18, True), (33, 384 * 128, 16, False), (63, 385 * 128 - 1, 19, True),
          (64, 512 * 128, 17, True), (48, 300 * 128 - 100, 20, False), (97, 300 * 128 - 9, 16, True), (127, 330 * 128, 18, True), (128, 384 * 128, 16, True)]
# beside them: 65 to 96 tokens, more panels, and lifted rows, on tiles of 128 x 128 or 256 x 256
BESIDE = [(65, 300 * 128 - 9, 16, True), (96, 384 * 128, 17, True), (97, 385 * 128 - 1, 17, True), (128, 512 * 128, 16, True), (100, 300 * 128, 16, False)]


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("M,O,units,fused", SHAPES + BESIDE)
def test_fragments_and_token_tiles(dtype, M, O, units, fused):
    _linear(M, O, _rows(units, 4, dtype, fused), 4, dtype, fused, False, M)


# packed weights of 80 MB and more, which are loaded non-temporally for up to 64 tokens, and of 256 MB and more for up to 128
@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("M,units", [(3, 22), (50, 22), (100, 22), (100, 70)])
def test_weights_larger_than_the_cache_keeps(dtype, M, units):
    _linear(M, 257 * 128 - 5, _rows(units, 4, dtype, True), 4, dtype, True, False, M)


@pytest.mark.parametrize("dtype", ["i8", "fp16"])
@pytest.mark.parametrize("M,pad_x,pad_y", [(5, 16, 1), (40, 128, 8), (100, 48, 4)])
def test_rows_with_gaps(dtype, M, pad_x, pad_y):
    O, K = 290 * 128 - 5, 128 * 16 // (1 if dtype == "i8" else 2)
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


# a workgroup per panel: fewer units than the ring holds to several rings, one range and several, ranges of unlike length
@pytest.mark.parametrize("dtype,N", [("i8", 4), ("bf16", 4), ("fp8", 3), ("fp16", 5)])
@pytest.mark.parametrize("M,O,units,with_ws", [(1, 129 * 128 - 5, 16, False), (31, 200 * 128, 21, False), (8, 192 * 128 + 4, 1, False), (32, 256 * 128, 3, False),
                                               (17, 192 * 128, 6, False), (1, 300, 131, True), (9, 4096, 65, True), (32, 1000, 160, True)])
def test_panels(dtype, N, M, O, units, with_ws):
    for fused in ([True, False] if N == 4 else [False]):
        _linear(M, O, _rows(units, N, dtype, fused), N, dtype, fused, with_ws, M)
