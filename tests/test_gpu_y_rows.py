"""Rows of Y that start anywhere, in the kernels that store a lane's channels as they are: every start within a 16-byte line, row lengths that leave none to all of a
lane's channels of the last panel, nothing written beside the rows.  Against a product in 64 bits; operands are small integers, so every partial sum is exact."""
import pytest
import torch

from paper_2603_05232_amd import binding

pytestmark = pytest.mark.gpu

# tokens, channels, units per row: 64-token and 128-token tiles, weight stream, small tiles of 32 and 64 channels
MID = [(33, 727, 1), (64, 300, 2), (40, 1001, 2), (300, 60 * 128 - 5, 12)]
WIDE = [(8, 140 * 128 - 3, 16), (64, 260 * 128 - 9, 16)]
SMALL = [(40, 6 * 128 - 5, 9), (17, 130, 5), (150, 20 * 128 - 120, 9), (256, 42 * 128 - 64, 9), (49, 727, 3)]


@pytest.mark.parametrize("dtype", ["i8", "fp16"])
@pytest.mark.parametrize("start,gap", [(0, 1), (1, 0), (2, 2), (3, 5), (4, 4), (7, 1), (8, 8)])
@pytest.mark.parametrize("M,O,units", MID + WIDE + SMALL)
def test_rows_anywhere(dtype, M, O, units, start, gap):
    K = 128 * units // (1 if dtype == "i8" else 2)
    td = torch.int8 if dtype == "i8" else torch.float16
    gen = torch.Generator(device="cuda").manual_seed(start + gap)
    X = torch.randint(-3, 4, (M, K), generator=gen, device="cuda").to(td)
    W = torch.where(torch.arange(K, device="cuda") % 8 < 6, torch.randint(-3, 4, (O, K), generator=gen, device="cuda"), 0)
    one = torch.ones(max(M, O), device="cuda") if dtype == "i8" else None
    wv, wm = binding.slide_decompose_fused(W.to(td), 4, dtype)
    out = torch.full((M + 1, start + O + gap), 7.0, dtype=torch.bfloat16, device="cuda")
    binding.slide_sparse_gemm_fused(X, None if one is None else one[:M], wv, wm, None if one is None else one[:O], O, K, 4, dtype, out=out[:M, start:start + O])
    assert torch.equal(out[:M, start:start + O], (X.double() @ W.double().T).bfloat16())
    assert bool((out[:M, :start] == 7.0).all()) and bool((out[:M, start + O:] == 7.0).all()) and bool((out[M] == 7.0).all())
