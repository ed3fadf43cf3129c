"""act_lift_quant on rows that start off a 16-byte line or end within one: the codes, the scales and the zeros behind the
row against the oracle, bit by bit, with values around the row that would change them if they were taken in."""
import numpy as np
import pytest
import torch

from oracle import slide_oracle as so
from paper_2603_05232_amd import binding, synth

from test_gpu_parity import check_lifted, dev, host

pytestmark = pytest.mark.gpu


# K: less than one vector, around the lengths up to which rows are loaded by elements (256, 512), around the widths of the launch choices (4 x 256, 4 x 512, 5 x 1024 vectors of 4 or 8 elements; the
# longest 8-bit rows that LDS holds), ends at every place within a line
@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("act", ["fp32", "bf16"])
@pytest.mark.parametrize("N,M,K,first,pad", [(4, 3, 1, 0, 2), (2, 4, 3, 1, 1), (4, 9, 7, 3, 0), (5, 9, 64, 5, 3), (3, 9, 256, 2, 1), (4, 9, 257, 1, 0), (2, 9, 258, 7, 3), (5, 9, 512, 3, 1), (3, 9, 513, 6, 0), (4, 9, 519, 0, 2), (3, 9, 1003, 2, 1), (2, 9, 1021, 7, 0),
                                             (8, 5, 4093, 6, 2), (4, 5, 4097, 1, 0), (7, 3, 8190, 3, 3), (6, 3, 8195, 4, 1), (4, 2, 16385, 0, 1),
                                             (3, 2, 20479, 2, 0), (5, 2, 32000, 3, 2), (4, 2, 65430, 1, 1)])
def test_rows_off_a_line(dtype, act, N, M, K, first, pad):
    if dtype in ("bf16", "fp16") and K > 32000:
        pytest.skip("the 16-bit row does not fit the LDS: refused")
    X = synth.activations(M, K, seed=K + N, n_outliers=min(4, K // 8))
    X[-1] = 0.0
    wide = np.full((M, first + K + pad), 1000.0 * np.abs(X).max() + 1.0, dtype=np.float32)
    wide[:, first:first + K] = X
    if act == "bf16":
        bits = so.bf16_bits(wide)
        X = so.bf16_to_f32(bits)[:, first:first + K]
        x = dev(bits.view(np.int16)).view(torch.bfloat16)[:, first:first + K]
    else:
        x = dev(wide)[:, first:first + K]
    exp, s = so.act_lift_quant(np.ascontiguousarray(X), N, dtype)
    got, gs = binding.act_lift_quant(x, N, dtype)
    check_lifted(got, exp, dtype)
    if dtype in ("i8", "fp8"):
        assert np.array_equal(host(gs), s)


def test_rows_off_a_line_smallest_scale():
    """The scale's reciprocal overflows (absmax below 127 / FLT_MAX): the zeros behind the row stay zeros."""
    X = np.zeros((2, 41), dtype=np.float32)
    X[:, ::3] = 1e-40
    exp, s = so.act_lift_quant(X, 4, "bf16")
    got, _ = binding.act_lift_quant(dev(X), 4, "bf16")
    check_lifted(got, exp, "bf16")
    q, _ = binding.act_lift_quant(dev(X), 4, "i8")
    assert not host(q)[:, 72:].any()                     # K' = 6 blocks x 12 = 72
