"""The 128-channel tile kernels at the edges of their token tiles (32, 64, 128), of their rings (one unit to several rings)
and of split k ranges, against a product in 64 bits.  Operands are small integers, so every partial sum is exact in all types."""
import pytest
import torch

from paper_2603_05232_amd import binding

pytestmark = pytest.mark.gpu


def _linear(M, O, K, N, dtype, fused, with_ws, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randint(-3, 4, (M, K), generator=gen, device="cuda")
    W = torch.randint(-3, 4, (O, K), generator=gen, device="cuda")
    X[:, 0] = 3                                                         # full scale present in every row: the codes are the integers times a constant
    if dtype in ("i8", "fp8"):
        td = torch.int8
        Wq = torch.where(torch.arange(K, device="cuda") % (2 * N) < 2 * N - 2, W, 0).to(td)
        Xq = X.to(td)
        s_x = torch.rand(M, generator=gen, device="cuda") + 0.5
        s_w = torch.rand(O, generator=gen, device="cuda") + 0.5
    else:
        td = torch.bfloat16 if dtype == "bf16" else torch.float16
        Wq = torch.where(torch.arange(K, device="cuda") % (2 * N) < 2 * N - 2, W, 0).to(td)
        Xq, s_x, s_w = X.to(td), None, None
    acc = (Xq.double() @ Wq.double().T).float()
    ref = (acc if s_x is None else (acc * s_x[:, None]) * s_w[None, :]).bfloat16()
    es = Xq.element_size()
    if fused:
        wv, wm = binding.slide_decompose_fused(Wq, N, dtype)
        row = K
        A = Xq
    else:
        wv, wm = binding.slide_decompose(Wq, N, dtype)
        row = binding.slide_lifted_ld(K, N, dtype)
        g = torch.arange(row // 4, device="cuda")
        src = (2 * N * (g // (N - 1)) + 2 * (g % (N - 1)))[:, None] + torch.arange(4, device="cuda")
        keep = (g[:, None] < -(-K // (2 * N)) * (N - 1)) & (src < K)
        A = torch.where(keep.reshape(-1), Xq[:, torch.where(keep, src, 0).reshape(-1)], torch.zeros((), dtype=td, device="cuda"))
    ws = None
    if with_ws:
        ws = torch.full((max(16, binding.slide_gemm_workspace_bytes(M, O, row, dtype)),), 0xFF, dtype=torch.uint8, device="cuda")
    out = torch.full((M + 1, O), 7.0, dtype=torch.bfloat16, device="cuda")
    if fused:
        binding.slide_sparse_gemm_fused(A, s_x, wv, wm, s_w, O, K, N, dtype, out=out[:M], workspace=ws)
    else:
        binding.slide_sparse_gemm(A.contiguous(), s_x, wv, wm, s_w, O, dtype, out=out[:M], workspace=ws)
    assert torch.equal(out[:M].view(torch.int16), ref.view(torch.int16))
    assert bool((out[M] == 7.0).all())                                 # nothing beyond the last token


# panels alone fill the chip: 192 panels and more, unsplit; 1 .. 18 units cover every state of the rings
@pytest.mark.parametrize("M", [1, 32, 33, 64])
@pytest.mark.parametrize("units", [1, 2, 3, 4, 5, 7, 8, 9, 10, 18])
def test_wide_layers_of_few_tokens(M, units):
    _linear(M, 192 * 128 - 5, 128 * units, 4, "i8", True, False, units)


# one workgroup per compute unit or several, split or not, tokens at the edges of the tiles, 16-bit and lifted forms
@pytest.mark.parametrize("dtype", ["i8", "bf16", "fp16"])
@pytest.mark.parametrize("M,O,units,N,fused", [(1, 520, 72, 4, True), (31, 130, 65, 4, True), (32, 384, 50, 4, True), (33, 260, 48, 4, True), (64, 1100, 57, 4, True),
                                               (65, 128, 9, 4, True), (128, 300, 1, 4, True), (129, 640, 17, 4, True), (200, 4224, 6, 4, True), (300, 10000, 3, 4, True),
                                               (4, 128, 66, 3, False), (40, 200, 52, 5, False), (127, 256, 33, 8, False), (257, 1000, 5, 2, False)])
def test_token_tiles_and_split_ranges(dtype, M, O, units, N, fused):
    es = 1 if dtype == "i8" else 2
    K = 128 * units // es
    if not fused:
        K = K * N // (2 * (N - 1)) - 3
    _linear(M, O, K, N, dtype, fused, True, M)


# one round of 256 x 256 tiles and a small rest of the channels on 128 x 128 tiles (256 compute units: 13056 + 500 channels)
@pytest.mark.parametrize("dtype,N,fused", [("i8", 4, True), ("bf16", 4, True), ("i8", 3, False), ("fp16", 5, False)])
def test_rest_of_a_round(dtype, N, fused):
    es = 1 if dtype == "i8" else 2
    K = 3 * 128 // es
    _linear(1100, 13556, K if fused else K * N // (2 * (N - 1)) - 3, N, dtype, fused, False, N)
