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
    if dtype in ("i8", "fp8"):
        def enc(a):                                                     # -3 .. 3 are e4m3 values
            return a.to(torch.int8) if dtype == "i8" else a.float().to(torch.float8_e4m3fn).view(torch.uint8)
        td = torch.int8 if dtype == "i8" else torch.uint8
        W = torch.where(torch.arange(K, device="cuda") % (2 * N) < 2 * N - 2, W, 0)
        Xq, Wq = enc(X), enc(W)
        s_x = torch.rand(M, generator=gen, device="cuda") + 0.5
        s_w = torch.rand(O, generator=gen, device="cuda") + 0.5
    else:
        td = torch.bfloat16 if dtype == "bf16" else torch.float16
        W = torch.where(torch.arange(K, device="cuda") % (2 * N) < 2 * N - 2, W, 0)
        Xq, Wq, s_x, s_w = X.to(td), W.to(td), None, None
    acc = (X.double() @ W.double().T).float()
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


# 192 panels, unsplit: one workgroup per compute unit (256 of them), the weight stream with a ring of four units (32 tokens) and tiles of 64 tokens with a
# ring of four units
@pytest.mark.parametrize("M", [1, 32, 33, 64])
@pytest.mark.parametrize("units", [1, 2, 3, 4, 5, 7, 8, 9, 10, 18])
def test_wide_layers_of_few_tokens(M, units):
    _linear(M, 192 * 128 - 5, 128 * units, 4, "i8", True, False, units)


def _rows(units, N, dtype, fused):
    """The longest row of `units` units of 128 bytes, less three elements where the form takes any length."""
    es = 1 if dtype in ("i8", "fp8") else 2
    return 128 * units // es if fused else 128 * units // es * N // (2 * (N - 1)) - 3


# 257 panels: workgroups share compute units.  Rings of four (32 tokens), three (64) and, for 128 tokens, two units in the
# pipeline (fused) and three without it (lifted), over row lengths from one unit to two rings and more
@pytest.mark.parametrize("dtype,N", [("i8", 4), ("bf16", 4), ("fp8", 3), ("fp16", 5)])
@pytest.mark.parametrize("M", [1, 32, 33, 64, 65, 128])
@pytest.mark.parametrize("units", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10])
def test_rings_of_shared_compute_units(dtype, N, M, units):
    for fused in ([True, False] if N == 4 else [False]):
        _linear(M, 257 * 128 - 5, _rows(units, N, dtype, fused), N, dtype, fused, False, units)


# the same with more than a quarter of the compute units shared and rows long enough for the pipeline of three (lifted) or
# two units (fused); three, nine and ten token tiles, the last two in two bands
SHARED = [("i8", 100, 321 * 128 - 3, 32, 4, False), ("bf16", 100, 322 * 128, 33, 4, False), ("fp8", 128, 330 * 128, 34, 3, False), ("fp16", 1100, 4700, 35, 5, False),
          ("i8", 1250, 3900, 9, 4, False), ("bf16", 1100, 3700, 7, 4, False), ("i8", 300, 130 * 128 - 3, 12, 4, True), ("bf16", 300, 130 * 128, 13, 4, True),
          ("i8", 1100, 52 * 128, 24, 4, True), ("fp16", 1100, 52 * 128 - 5, 25, 4, True), ("fp8", 1100, 55 * 128, 26, 4, True)]
# at most one tile of 128 channels x 256 tokens per compute unit: those
SHARED_NARROW = [("i8", 1250, 4200, 12, 4, True), ("bf16", 1100, 4700, 13, 4, True)]


@pytest.mark.parametrize("dtype,M,O,units,N,fused", SHARED + SHARED_NARROW)
def test_shared_pipelines_and_bands(dtype, M, O, units, N, fused):
    _linear(M, O, _rows(units, N, dtype, fused), N, dtype, fused, False, units)


# Both sides of lines of the kernel choice for sparse calls, for 256 compute units: tiles (320, 448, 512) and units
# per row (12 and 24 fused, 24 and 48 lifted) between 128 x 128 and 256 x 256 tiles; panels (128 and 192) between the few-token kernel and the weight
# stream of 32 tokens, on either side of half as many panels as compute units with 64 tokens (small tiles on both); rows (1 token 64 units, 32 to 64 tokens 48) between
# unsplit kernels and, with the workspace, split ones; a rest of a round of exactly one tile per compute unit and of one panel more, and, fused, of up to one 128 x 256
# tile (16 units and more).
@pytest.mark.parametrize("M,O,units,ws", [(65, 128 * 320, 3, False), (65, 128 * 321, 11, False), (65, 128 * 321, 12, False), (65, 128 * 321, 23, False),
                                          (65, 128 * 321, 24, False), (65, 128 * 448, 12, False), (65, 128 * 449, 23, False), (65, 128 * 449, 24, False),
                                          (65, 128 * 449, 47, False), (65, 128 * 449, 48, False), (65, 128 * 512, 48, False), (65, 128 * 513, 48, False),
                                          (15, 128 * 191, 3, False), (15, 128 * 192, 3, False), (16, 128 * 127, 3, False), (16, 128 * 128, 3, False),
                                          (64, 128 * 127, 3, False), (64, 128 * 128, 3, False), (1, 500, 63, True), (1, 500, 64, True), (32, 500, 47, True),
                                          (32, 500, 48, True), (33, 500, 47, True), (33, 500, 48, True), (64, 500, 47, True), (64, 500, 48, True),
                                          (1000, 16384 + 4096, 3, False), (1000, 16384 + 4097, 3, False),
                                          (8100, 2048 + 1000, 15, False), (8100, 2048 + 1000, 16, False), (8100, 2048 + 1100, 16, False)])
@pytest.mark.parametrize("fused", [True, False])
def test_lines_of_the_kernel_choice(M, O, units, ws, fused):
    _linear(M, O, _rows(units, 4, "i8", fused), 4, "i8", fused, ws, units)


# split rows and unsplit ones (of up to 33 units: small tiles and 128 x 128 ones), tokens at the edges of the tiles, 16-bit and lifted forms
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


# up to 32 tokens with two groups of wavefronts (lifted rows on half to two thirds as many panels as compute units, 12 units and more, M < 16: 16):
# ranges of odd and even length, from one ring and less for each group to several, the fewest and the most panels, weights of 80 MB and more
TWO_GROUPS = [(16, 128 * 128, 12), (31, 129 * 128 - 5, 13), (32, 170 * 128, 14), (1, 129 * 128, 16), (9, 170 * 128 - 100, 17), (15, 140 * 128 + 4, 33),
              (20, 150 * 128, 41), (32, 160 * 128 - 1, 54)]


@pytest.mark.parametrize("dtype,N", [("i8", 4), ("fp8", 3), ("bf16", 4), ("fp16", 5)])
@pytest.mark.parametrize("M,O,units", TWO_GROUPS)
def test_two_groups_of_wavefronts(dtype, N, M, O, units):
    _linear(M, O, _rows(units, N, dtype, False), N, dtype, False, False, units)


# up to 32 tokens by the weight stream: odd and even rows, one range (130 and 192 panels) and several (few panels and long rows)
STREAM = [(1, 192 * 128 - 5, 2, False), (32, 192 * 128, 3, False), (17, 130 * 128, 9, False), (1, 300, 131, True), (32, 1000, 160, True), (9, 512, 97, True)]


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("M,O,units,with_ws", STREAM)
def test_stream_of_a_panel(dtype, fused, M, O, units, with_ws):
    N = 4
    es = 1 if dtype in ("i8", "fp8") else 2
    K = 128 * units // es if fused else 128 * units // es * N // (2 * (N - 1)) // (2 * N) * (2 * N)
    _linear(M, O, max(K, 2 * N), N, dtype, fused, with_ws, units)


# the same on half as many panels as compute units, unlifted rows of more than 42 units
LONG_ROWS = [(16, 128 * 128, 43), (25, 128 * 128 - 5, 68), (32, 128 * 128, 97)]


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("M,O,units", LONG_ROWS)
def test_stream_of_half_as_many_panels(dtype, M, O, units):
    _linear(M, O, _rows(units, 4, dtype, True), 4, dtype, True, False, units)


# the few-token kernel: rows of up to three units for 17 to 32 tokens, on few panels and on up to half as many as compute units; up to 16 tokens short rows on 65 to 128
# panels and, a workgroup for two fragments, on up to 191
FEW_TOKENS = [(17, 300, 1), (32, 63 * 128 - 5, 3), (20, 64 * 128, 2), (31, 127 * 128 - 3, 3), (5, 65 * 128, 11), (16, 100 * 128 - 4, 9), (15, 127 * 128, 8),
              (1, 100 * 128, 11), (15, 129 * 128, 3), (3, 160 * 128 - 1, 8), (15, 191 * 128, 15)]


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("M,O,units", FEW_TOKENS)
def test_few_tokens(dtype, fused, M, O, units):
    _linear(M, O, _rows(units, 4, dtype, fused), 4, dtype, fused, False, units)


# packed weights of 80 MB and more, which are loaded non-temporally: unsplit panels and split rows, the weight stream (3 tokens) and tiles of 64 tokens
# (8-bit types; 16-bit ones from 256 MB on)
@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("M", [3, 50])
@pytest.mark.parametrize("O,units", [(192 * 128 + 4, 29), (24 * 128, 230)])
def test_weights_larger_than_the_cache_keeps(dtype, M, O, units):
    _linear(M, O, _rows(units, 4, dtype, True), 4, dtype, True, True, M)


# split rows by the number of ranges that the reduce kernel adds (eight at a time, the last one to four of them by four or two): a full
# batch and 1, 2, 3, 4, 5 or 8 more, two full batches and more, many; tiles of 32, 64 and 128 tokens
RANGES = [(M, 300, 8 * S, S) for M in (5, 40) for S in (8, 9, 10, 11, 12, 13, 16, 17, 21)] + [(33, 300, 48, 6), (100, 128, 300, 34)]


@pytest.mark.parametrize("dtype,fused", [("i8", True), ("bf16", False)])
@pytest.mark.parametrize("M,O,units,S", RANGES)
def test_numbers_of_ranges(dtype, fused, M, O, units, S):
    _linear(M, O, _rows(units, 4, dtype, fused), 4, dtype, fused, True, S)


# split rows on 32 tiles (a workgroup of the reduce kernel for each block of 32 channels x 32 tokens) and on more (one for all blocks of a wavefront), of 64 and 128
# tokens, with tokens and channels missing in the last tile
BLOCKS = [(64, 32 * 128, 64), (50, 33 * 128 - 5, 64), (128, 32 * 128 - 3, 48), (70, 33 * 128, 48), (200, 16 * 128, 48), (200, 17 * 128 - 4, 48)]


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("M,O,units", BLOCKS)
def test_blocks_of_the_reduce_kernel(dtype, fused, M, O, units):
    _linear(M, O, _rows(units, 4, dtype, fused), 4, dtype, fused, True, M)


# the same, each with its limit in MB: tiles of 32 tokens on shared compute units, tiles of 64 on shared ones, and with one each in 8-bit and in 16-bit types
LARGE = [(3, 513 * 128, 16, True, 80), (30, 513 * 128 - 5, 17, False, 80), (50, 513 * 128, 35, True, 256), (40, 520 * 128 - 3, 52, False, 256),
         (50, 200 * 128, 28, True, 80), (33, 224 * 128 - 4, 48, False, 80), (64, 250 * 128, 72, True, 256), (60, 256 * 128, 104, False, 256)]


@pytest.mark.parametrize("dtype", ["i8", "bf16"])
@pytest.mark.parametrize("M,O,units,fused,limit", LARGE)
def test_large_weights(dtype, M, O, units, fused, limit):
    _linear(M, O, _rows(units, 4, dtype, fused), 4, dtype, fused, False, M)
