"""act_lift_quant at the lengths and token counts where the threads of a row change (one workgroup per compute unit or more, 256 of them;
256, 1024 and 2048 vectors of 4 or 8 elements, and one more): first, middle and last row against the oracle, bit by bit, whole lines and rows off one."""
import numpy as np
import pytest
import torch

from oracle import slide_oracle as so
from paper_2603_05232_amd import binding, synth

from test_gpu_parity import check_lifted, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("act", ["fp32", "bf16"])
@pytest.mark.parametrize("M", [256, 257])
@pytest.mark.parametrize("N,vectors,extra", [(2, 256, 0), (4, 257, 0), (2, 1024, 0), (4, 1024, 0), (5, 1025, 0), (4, 2048, 0), (3, 2049, 0), (4, 700, 1), (2, 1500, 3)])
def test_edges_of_the_thread_counts(dtype, act, M, N, vectors, extra):
    K = vectors * (4 if act == "fp32" else 8) + extra
    X = synth.activations(M, K, seed=K + N, n_outliers=4)
    if act == "bf16":
        bits = so.bf16_bits(X)
        X = so.bf16_to_f32(bits)
        x = dev(bits.view(np.int16)).view(torch.bfloat16)
    else:
        x = dev(X)
    rows = [0, M // 2, M - 1]
    exp, s = so.act_lift_quant(np.ascontiguousarray(X[rows]), N, dtype)
    got, gs = binding.act_lift_quant(x, N, dtype)
    check_lifted(got[rows], exp, dtype)
    if dtype in ("i8", "fp8"):
        assert np.array_equal(host(gs)[rows], s)
