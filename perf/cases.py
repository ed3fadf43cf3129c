"""The work a user of this library has it do, as cases that can be timed and whose outputs can be compared.

Two kinds of case.  "linear": the online path of a (2N-2):2N sparse linear layer, or of the four linear layers of one
transformer block one after the other (qkv, o, gate_up, down): per-token quantisation, then the sparse GEMM with the
workspace it asks for.  path "fused" quantises alone and lifts inside the GEMM (6:8 with whole 128-byte rows), path
"lifted" quantises and lifts, then multiplies (every pattern, every K).  "pack": the offline path of a weight matrix,
magnitude pruning + per-channel quantisation, then decomposition and packing for the GEMM of that path.

Weights, activations and shapes are those of synth.py (Gaussian, a few outlier channels x20), drawn on the GPU."""
import math

import torch

from paper_2603_05232_amd import binding, synth

MODELS = {"qwen25_7b": synth.QWEN25_7B, "llama3_8b": synth.LLAMA3_8B}
ACT_DTYPE = {"fp32": torch.float32, "bf16": torch.bfloat16}
ELEM_SIZE = {"i8": 1, "fp8": 1, "bf16": 2, "fp16": 2}


def listed():
    def linear(name, path, N, dtype, act, M, **layers):
        return {"name": name, "kind": "linear", "path": path, "N": N, "dtype": dtype, "act": act, "M": M, **layers}

    return [
        # one small layer, the library's anchor example: nothing but launches and host calls
        linear("small_m16_i8", "lifted", 4, "i8", "fp32", 16, K=512, O=512),
        # decode of one sequence: every weight of a block is streamed once for one token
        linear("decode_m1_i8", "fused", 4, "i8", "bf16", 1, model="qwen25_7b"),
        # decode of a small batch with unscaled 16-bit operands
        linear("decode_m16_bf16", "fused", 4, "bf16", "bf16", 16, model="qwen25_7b"),
        # decode of a served batch, the smallest token count the method's own end-to-end runs use, lifted path
        linear("batch_m64_fp8_lifted", "lifted", 4, "fp8", "bf16", 64, model="llama3_8b"),
        # a large decode batch or a short prompt
        linear("batch_m256_i8", "fused", 4, "i8", "bf16", 256, model="qwen25_7b"),
        # a prompt of odd length through a layer whose width is no multiple of the pattern or of a cache line
        linear("ragged_m777_8of10_fp16", "lifted", 5, "fp16", "fp32", 777, K=5003, O=4099),
        # one chunk of a chunked prefill
        linear("chunk_m2048_fp8", "fused", 4, "fp8", "bf16", 2048, model="llama3_8b"),
        # the linears of a Llama-3-8B-shaped block over one sequence
        linear("block_m4096_i8", "fused", 4, "i8", "bf16", 4096, model="llama3_8b"),
        # prefill: the benchmark's step
        linear("prefill_m8192_i8", "fused", 4, "i8", "fp32", 8192, model="qwen25_7b"),
        # prefill with unscaled 16-bit operands
        linear("prefill_m8192_bf16", "fused", 4, "bf16", "bf16", 8192, model="qwen25_7b"),
        # another pattern of the family, which only the lifted path serves
        linear("prefill_m8192_4of6_i8", "lifted", 3, "i8", "fp32", 8192, K=6144, O=4096),
        # preparing the weights of a block for the fused path from a 16-bit checkpoint
        {"name": "pack_block_i8", "kind": "pack", "path": "fused", "N": 4, "dtype": "i8", "act": "bf16", "model": "qwen25_7b"},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MAX_FLOPS = 8192 * sum(K * O for _, K, O in synth.QWEN25_7B)     # a drawn linear: at most half the largest listed one
MAX_PACK = sum(K * O for _, K, O in synth.QWEN25_7B)


def draw(rng):
    """One layer of the ranges above: tokens 1..8192, K 256..18944, O 128..37888 (all spread over their logarithm), every
    operand type, activation type, pattern and path; a quarter of the draws prepare weights."""
    dtype = rng.choice(["i8", "i8", "fp8", "bf16", "fp16"])
    path = rng.choice(["fused", "fused", "lifted"])
    act = rng.choice(["fp32", "bf16"])
    per_line = 128 // ELEM_SIZE[dtype]
    pack = rng.random() < 0.25
    while True:
        K, O, M = _log_int(rng, 256, 18944), _log_int(rng, 128, 37888), _log_int(rng, 1, 8192)
        if path == "fused":
            N, K = 4, (K + per_line - 1) // per_line * per_line
        else:
            N = rng.choice([2, 3, 4, 4, 5, 6, 7, 8])
            if rng.random() < 0.7:                       # most widths are multiples of 128; the others stay as they come
                K = (K + 127) // 128 * 128
        if rng.random() < 0.7:
            O = (O + 63) // 64 * 64
        if K * O <= MAX_PACK and 2 * M * K * O <= MAX_FLOPS:
            break
    case = {"kind": "pack" if pack else "linear", "path": path, "N": N, "dtype": dtype, "act": act, "K": K, "O": O}
    if not pack:
        case["M"] = M
    return case


def _layers(case):
    return [(K, O) for _, K, O in MODELS[case["model"]]] if "model" in case else [(case["K"], case["O"])]


def _activations(gen, M, K, dtype):
    X = torch.randn((M, K), generator=gen, device="cuda", dtype=torch.float32)
    cols = torch.randperm(K, generator=gen, device="cuda")[: synth.n_outlier_columns(K)]
    X[:, cols] *= 20.0
    return X.to(dtype)


def _weights(gen, O, K, dtype):
    return torch.randn((O, K), generator=gen, device="cuda", dtype=torch.float32).mul_(0.02).to(dtype)


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    N, dtype, fused = case["N"], case["dtype"], case["path"] == "fused"
    src = ACT_DTYPE[case["act"]]
    layers = []
    if case["kind"] == "pack":
        for K, O in _layers(case):
            layers.append(_weights(gen, O, K, src))
        return {"case": case, "layers": layers}
    ws_bytes = 0
    for K, O in _layers(case):
        Wq, s_w = binding.slide_prune_quant(_weights(gen, O, K, src), N, dtype)
        w_vals, w_meta = (binding.slide_decompose_fused if fused else binding.slide_decompose)(Wq, N, dtype)
        row = K if fused else binding.slide_lifted_ld(K, N, dtype)
        ws_bytes = max(ws_bytes, binding.slide_gemm_workspace_bytes(case["M"], O, row, dtype))
        layers.append({"K": K, "O": O, "X": _activations(gen, case["M"], K, src), "w_vals": w_vals, "w_meta": w_meta, "s_w": s_w})
    ws = torch.empty((ws_bytes,), dtype=torch.uint8, device="cuda") if ws_bytes else None
    return {"case": case, "layers": layers, "workspace": ws}


def run(state):
    case = state["case"]
    N, dtype, fused = case["N"], case["dtype"], case["path"] == "fused"
    outs = []
    if case["kind"] == "pack":
        for W in state["layers"]:
            Wq, s_w = binding.slide_prune_quant(W, N, dtype)
            outs.append((Wq, s_w) + (binding.slide_decompose_fused if fused else binding.slide_decompose)(Wq, N, dtype))
        return outs
    ws = state["workspace"]
    for L in state["layers"]:
        if fused:
            Xq, s_x = binding.act_lift_quant(L["X"], 2, dtype)
            Y = binding.slide_sparse_gemm_fused(Xq, s_x, L["w_vals"], L["w_meta"], L["s_w"], L["O"], L["K"], N, dtype, workspace=ws)
        else:
            XL, s_x = binding.act_lift_quant(L["X"], N, dtype)
            Y = binding.slide_sparse_gemm(XL, s_x, L["w_vals"], L["w_meta"], L["s_w"], L["O"], dtype, workspace=ws)
        outs.append(Y)
    return outs


def work(case):
    """linear: activations, stored weights (the values and a 2-bit position for each) and scales read once, Y written
    once; two operations per token and stored weight.  pack: the weight matrix read once; the quantised matrix, its
    scales and the packed form written once."""
    N, es, src = case["N"], ELEM_SIZE[case["dtype"]], 4 if case["act"] == "fp32" else 2
    nbytes = flops = 0
    for K, O in _layers(case):
        kept = K * (N - 1) / N
        packed = O * kept * (es + 0.25)
        if case["kind"] == "pack":
            nbytes += O * K * (src + es) + packed + (4 * O if es == 1 else 0)
        else:
            M = case["M"]
            nbytes += M * K * src + packed + 2 * M * O + (4 * O if es == 1 else 0)
            flops += 2 * M * O * kept
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Weight preparation and INT8 are exact by definition (one correctly rounded operation at a time, int32 sums).
    if case["kind"] == "pack" or case["dtype"] == "i8":
        return "exact"
    # Measured against the product in 64 bits rounded once to bf16 (K up to 18944): rel 2.2e-4 to 2.6e-4 for fp8, whose
    # matrix instructions keep 14 bits below a group's largest product, 2e-5 to 5e-5 for bf16 / fp16; the largest single
    # difference is one bf16 step (7.8e-3).  Four times that, plus one output in a small result rounded the other way.
    outputs = case["M"] * sum(O for _, O in _layers(case))
    return {"rel": (1e-3 if case["dtype"] == "fp8" else 2e-4) + 2.0 ** -7 / math.sqrt(outputs), "max": 1.6e-2}
