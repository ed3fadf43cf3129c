"""GPU parity at the full sizes of the benchmark configurations, in the launch configuration bench.py
times: the whole hot path runs on the full tensors, and the CPU oracle recomputes a random sample of
output elements (whole tokens x whole channels are independent of the rest: quantisation is per token
and per channel, pruning per channel).  INT8 must be bit-exact; in addition the sparse and the dense
path must agree on every element of the full output."""
import numpy as np
import pytest
import torch

from oracle import slide_oracle as so
from paper_2603_05232_amd import binding, synth
from test_gpu_parity import dev, host, bits16, from_dev_q, _float_gemm_check

pytestmark = pytest.mark.gpu
N_SAMPLE = 96


def _run_and_sample(M, K, O, N, dtype, seed, use_workspace=False):
    X = synth.activations(M, K, seed)
    W = synth.weights(O, K, seed)
    Xd, Wd = dev(X), dev(W)
    Wq, s_w = binding.slide_prune_quant(Wd, N, dtype)
    del Wd
    w_vals, w_meta, viol = binding.slide_decompose(Wq, N, dtype, count_violations=True)
    XL, s_x = binding.act_lift_quant(Xd, N, dtype)
    ws_s = ws_d = None
    if use_workspace:                                            # k range split over workgroups where the library would
        ns, nd = binding.slide_gemm_workspace_bytes(M, O, XL.shape[1], dtype), binding.slide_gemm_workspace_bytes(M, O, K, dtype)
        assert ns > 0 and nd > 0
        ws_s = torch.empty((ns,), dtype=torch.uint8, device=XL.device)
        ws_d = torch.empty((nd,), dtype=torch.uint8, device=XL.device)
    Y = binding.slide_sparse_gemm(XL, s_x, w_vals, w_meta, s_w, O, dtype, workspace=ws_s)
    Y2 = binding.slide_sparse_gemm(XL, s_x, w_vals, w_meta, s_w, O, dtype, workspace=ws_s)
    Xq, s_x2 = binding.act_lift_quant(Xd, 2, dtype)
    Yd = binding.dense_gemm(Xq, s_x2, Wq, s_w, dtype, workspace=ws_d)
    assert int(host(viol)[0]) == 0
    assert torch.equal(Y, Y2)                                    # deterministic from launch to launch
    Yf = None
    if N == 4 and (K * Xq.element_size()) % 128 == 0:            # the same layer with the lifting applied inside the GEMM
        fw_vals, fw_meta = binding.slide_decompose_fused(Wq, N, dtype)
        Yf = binding.slide_sparse_gemm_fused(Xq, s_x2, fw_vals, fw_meta, s_w, O, K, N, dtype)
        assert torch.equal(Yf, binding.slide_sparse_gemm_fused(Xq, s_x2, fw_vals, fw_meta, s_w, O, K, N, dtype))
        del fw_vals, fw_meta
    rng = np.random.default_rng(seed + 12345)
    rows = np.sort(rng.choice(M, size=min(M, N_SAMPLE), replace=False))
    cols = np.sort(rng.choice(O, size=min(O, N_SAMPLE), replace=False))
    if M > 1:
        rows[-1] = M - 1                                         # the last token and channel: tile tails
    cols[-1] = O - 1
    ref = so.linear_reference(X[rows], W[cols], N, dtype)
    ri, ci = torch.from_numpy(rows).to(Y.device), torch.from_numpy(cols).to(Y.device)
    sample = lambda T: bits16(T[ri][:, ci].contiguous())
    # operands the sample depends on
    assert np.array_equal(from_dev_q(Wq[ci].contiguous(), dtype), ref["Wq"])
    assert np.array_equal(from_dev_q(Xq[ri].contiguous(), dtype), ref["Xq"])
    assert np.array_equal(from_dev_q(XL[ri].contiguous(), dtype), so.lift(ref["Xq"], N))
    if Yf is not None:                                           # checked here so that every caller covers the fused path
        if dtype == "i8":
            assert np.array_equal(sample(Yf), ref["Y"])
            assert torch.equal(Yf, Yd)
        else:
            _float_gemm_check(sample(Yf), ref, dtype)
    return Y, Yd, sample, ref


@pytest.mark.parametrize("name,K,O", synth.QWEN25_7B)
def test_qwen25_7b_int8_m8192(name, K, O):
    Y, Yd, sample, ref = _run_and_sample(8192, K, O, 4, "i8", seed=len(name))
    assert np.array_equal(sample(Y), ref["Y"])
    assert torch.equal(Y, Yd)


@pytest.mark.parametrize("N,K,O", synth.PATTERN_SWEEP)
def test_pattern_sweep_int8_m8192(N, K, O):
    Y, Yd, sample, ref = _run_and_sample(8192, K, O, N, "i8", seed=N)
    assert np.array_equal(sample(Y), ref["Y"])
    assert torch.equal(Y, Yd)


@pytest.mark.parametrize("name,K,O", synth.LLAMA3_8B)
def test_llama3_8b_block_int8_m4096(name, K, O):
    Y, Yd, sample, ref = _run_and_sample(4096, K, O, 4, "i8", seed=10 + len(name))
    assert np.array_equal(sample(Y), ref["Y"])
    assert torch.equal(Y, Yd)


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("M", [1, 16, 128])
@pytest.mark.parametrize("name,K,O", synth.QWEN25_7B)
def test_qwen25_7b_small_m(dtype, M, name, K, O):
    Y, Yd, sample, ref = _run_and_sample(M, K, O, 4, dtype, seed=M)
    if dtype == "i8":
        assert np.array_equal(sample(Y), ref["Y"])
        assert torch.equal(Y, Yd)
    else:
        _float_gemm_check(sample(Y), ref, dtype)
        _float_gemm_check(sample(Yd), ref, dtype)


@pytest.mark.parametrize("dtype", ["fp8", "bf16", "fp16"])
@pytest.mark.parametrize("name,K,O", synth.QWEN25_7B)
def test_qwen25_7b_float_m8192(dtype, name, K, O):
    Y, Yd, sample, ref = _run_and_sample(8192, K, O, 4, dtype, seed=7)
    _float_gemm_check(sample(Y), ref, dtype)
    _float_gemm_check(sample(Yd), ref, dtype)


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16"])
@pytest.mark.parametrize("M", [128, 256])
@pytest.mark.parametrize("name,K,O", [synth.QWEN25_7B[0], synth.QWEN25_7B[3]])
def test_qwen25_7b_mid_m_with_workspace(dtype, M, name, K, O):
    """Token counts between decode and prefill, with a workspace: small unsplit tiles (qkv in 8-bit types), 128 x 128 tiles with the k range split (the others)."""
    Y, Yd, sample, ref = _run_and_sample(M, K, O, 4, dtype, seed=M + 1, use_workspace=True)
    if dtype == "i8":
        assert np.array_equal(sample(Y), ref["Y"])
        assert torch.equal(Y, Yd)
    else:
        _float_gemm_check(sample(Y), ref, dtype)
        _float_gemm_check(sample(Yd), ref, dtype)


@pytest.mark.parametrize("M,O", [(3, 40), (65, 16)])
def test_longest_rows_int8(M, O):
    """Rows at the documented maximum of the GEMMs (2^23 bytes; here K' = 65535 units of 128 bytes) on the
    kernels of 16 channels a workgroup (M = 3) and of small tiles (M = 65) without a workspace, on the weight stream and 128 x 128 tiles
    in split rows with one: 32-bit lane offsets and unit counters at their limits.  Operands are generated quantised (the lifting kernel keeps a row in
    LDS and stops at 64 KiB); the oracle lifts and multiplies."""
    from oracle import gemm_ref
    N = 4
    K = 65535 * 128 * 2 // 3                                   # K' = 1.5 K = 65535 * 128
    assert K % 8 == 0 and so.lifted_k(K, N) == 65535 * 128 == binding.slide_lifted_ld(K, N, "i8")
    rng = np.random.default_rng(M)
    Wq = rng.integers(-127, 128, size=(O, K), dtype=np.int8)
    Wq.reshape(O, K // 8, 8)[:, :, rng.permutation(8)[:2]] = 0    # two zeros per block of 8 (same positions everywhere)
    Wq.reshape(O, K // 8, 8)[:, ::3, 5] = 0                       # some blocks with three
    Xq = rng.integers(-127, 128, size=(M, K), dtype=np.int8)
    s_x = rng.uniform(0.001, 0.01, M).astype(np.float32)
    s_w = rng.uniform(1e-5, 1e-4, O).astype(np.float32)
    exp = so.epilogue(gemm_ref.gemm_i8_i64(Xq, Wq), s_x, s_w, "i8")
    w_vals, w_meta, viol = binding.slide_decompose(dev(Wq), N, "i8", count_violations=True)
    assert int(host(viol)[0]) == 0
    XL = dev(so.lift(Xq, N))
    Y = binding.slide_sparse_gemm(XL, dev(s_x), w_vals, w_meta, dev(s_w), O, "i8")
    assert np.array_equal(bits16(Y), exp)
    n = binding.slide_gemm_workspace_bytes(M, O, XL.shape[1], "i8")
    if n:
        ws = torch.empty((n,), dtype=torch.uint8, device=XL.device)
        assert np.array_equal(bits16(binding.slide_sparse_gemm(XL, dev(s_x), w_vals, w_meta, dev(s_w), O, "i8", workspace=ws)), exp)
    if K % 128 == 0:
        assert np.array_equal(bits16(binding.dense_gemm(dev(Xq), dev(s_x), dev(Wq), dev(s_w), "i8")), exp)


@pytest.mark.parametrize("M,ldy_log2", [(70000, 16), (300, 21), (20, 21)])
def test_output_offsets_beyond_32_bits(M, ldy_log2):
    """Y with a row stride so large that element offsets exceed 2^32 (M = 70000, ldy = 2^16: 256 x 256 tiles) or byte
    offsets 2^31 (ldy = 2^21: 128 x 128 tiles and the few-token kernels): 64-bit addressing of the output, and nothing
    is written outside the result columns."""
    N, K, O = 4, 256, 64
    ldy = 1 << ldy_log2
    rng = np.random.default_rng(M)
    Wq = rng.integers(-127, 128, size=(O, K), dtype=np.int8)
    Wq.reshape(O, K // 8, 8)[:, :, [1, 6]] = 0
    Xq = rng.integers(-127, 128, size=(M, K), dtype=np.int8)
    s_x = rng.uniform(0.01, 0.1, M).astype(np.float32)
    s_w = rng.uniform(1e-4, 1e-3, O).astype(np.float32)
    w_vals, w_meta = binding.slide_decompose(dev(Wq), N, "i8")
    XL = dev(so.lift(Xq, N))
    buf = torch.zeros((M, ldy), dtype=torch.bfloat16, device=XL.device)
    assert buf.numel() > 2 ** 32 or M < 2048
    binding.slide_sparse_gemm(XL, dev(s_x), w_vals, w_meta, dev(s_w), O, "i8", out=buf[:, :O])
    rows = np.unique(np.concatenate([rng.choice(M, size=min(M, 64), replace=False), [0, M - 1]]))
    exp = so.epilogue(so.gemm_exact(Xq[rows], Wq, "i8"), s_x[rows], s_w, "i8")
    ri = torch.from_numpy(rows).to(buf.device)
    assert np.array_equal(bits16(buf[ri][:, :O].contiguous()), exp)
    assert not bool(buf[ri][:, O:O + 4096].any())                          # columns beside the result stay zero
    total = buf[:, :O].float().abs().sum().item()
    assert abs(buf.float().abs().sum().item() - total) <= 1e-3 * total     # nothing was written anywhere else
    buf.zero_()
    binding.dense_gemm(dev(Xq), dev(s_x), dev(Wq), dev(s_w), "i8", out=buf[:, :O])
    assert np.array_equal(bits16(buf[ri][:, :O].contiguous()), exp)


@pytest.mark.parametrize("dtype", ["i8", "fp8"])
def test_two_persistent_rounds_full_output(dtype):
    """More 256 x 256 tiles than compute units (17 x 18 = 306; dense: a second persistent round with its tile renumbering, the
    next tile's first unit requested before the epilogue, scale parity; sparse: one round of 17 x 15, the channels behind it on 128 x
    128 tiles) with ragged edges and a short K, so that the CPU oracle can check EVERY output element of the sparse and of the dense kernel (not one against the other)."""
    from oracle import gemm_ref
    N, M, O, K = 4, 4300, 4400, 256
    rng = np.random.default_rng(11)
    if dtype == "i8":
        Wq = rng.integers(-127, 128, size=(O, K)).astype(np.int8)
        keep = np.argsort(rng.random((O, K // 8, 8)), axis=-1) < rng.integers(0, 7, size=(O, K // 8, 1))
        Wq = (Wq.reshape(O, K // 8, 8) * keep).reshape(O, K).astype(np.int8)
        Xq = rng.integers(-127, 128, size=(M, K)).astype(np.int8)
        s_x = rng.uniform(0.01, 0.1, M).astype(np.float32)
        s_w = rng.uniform(1e-4, 1e-3, O).astype(np.float32)
        exp = so.epilogue(gemm_ref.gemm_i8_i64(Xq, Wq), s_x, s_w, "i8")
        w_vals, w_meta = binding.slide_decompose(dev(Wq), N, "i8")
        Ys = binding.slide_sparse_gemm(dev(so.lift(Xq, N)), dev(s_x), w_vals, w_meta, dev(s_w), O, "i8")
        assert np.array_equal(bits16(Ys), exp)
        Yd = binding.dense_gemm(dev(Xq), dev(s_x), dev(Wq), dev(s_w), "i8")
        assert np.array_equal(bits16(Yd), exp)
    else:
        X = synth.activations(M, K, seed=3)
        W = synth.weights(O, K, seed=3)
        ref = so.linear_reference(X, W, N, dtype)
        Wq, s_w = binding.slide_prune_quant(dev(W), N, dtype)
        w_vals, w_meta = binding.slide_decompose(Wq, N, dtype)
        XL, s_x = binding.act_lift_quant(dev(X), N, dtype)
        _float_gemm_check(bits16(binding.slide_sparse_gemm(XL, s_x, w_vals, w_meta, s_w, O, dtype)), ref, dtype)
        Xq, s_x2 = binding.act_lift_quant(dev(X), 2, dtype)
        _float_gemm_check(bits16(binding.dense_gemm(Xq, s_x2, Wq, s_w, dtype)), ref, dtype)
        fw_vals, fw_meta = binding.slide_decompose_fused(Wq, N, dtype)
        _float_gemm_check(bits16(binding.slide_sparse_gemm_fused(Xq, s_x2, fw_vals, fw_meta, s_w, O, K, N, dtype)), ref, dtype)


def test_documented_limits():
    """Limits the header states: act_lift_quant keeps the quantised row in 64 KiB of LDS; dense_gemm wants whole
    128-byte rows while the sparse side pads ragged K itself."""
    x = torch.zeros((2, 65536), dtype=torch.float32, device="cuda:0")
    with pytest.raises(binding.SlideSparseError) as e:
        binding.act_lift_quant(x, 4, "i8")                                   # 65536 + 8 bytes of quantised row
    assert e.value.code == 3
    binding.act_lift_quant(x[:, :65536 - 128], 4, "i8")                      # just below the limit
    Xq = torch.zeros((4, 200), dtype=torch.int8, device="cuda:0")
    Wq = torch.zeros((128, 200), dtype=torch.int8, device="cuda:0")
    s = torch.ones((128,), dtype=torch.float32, device="cuda:0")
    with pytest.raises(binding.SlideSparseError) as e:
        binding.dense_gemm(Xq, s[:4], Wq, s, "i8")                           # K = 200 bytes is not a multiple of 128
    assert e.value.code == 3
    w_vals, w_meta = binding.slide_decompose(Wq, 4, "i8")                    # the sparse side pads K' = 300 to 384
    XL, s_x = binding.act_lift_quant(torch.zeros((4, 200), dtype=torch.float32, device="cuda:0"), 4, "i8")
    assert XL.shape[1] == 384
    assert not bool(binding.slide_sparse_gemm(XL, s_x, w_vals, w_meta, s, 128, "i8").any())
