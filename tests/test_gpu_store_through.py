"""Quantisation, lifting and pruning on either side of the lines between which they store through the L2 (pruning from 4 MB of output; the quantiser from 4 MB to 8, 16 or 32 MB,
by the length of the rows): the rows of one call are those of calls on a few rows each."""
import pytest
import torch

from paper_2603_05232_amd import binding

pytestmark = pytest.mark.gpu


# whole and ragged rows, from either type, lifted and not; the last MB with stores through the L2
ROWS = [("bf16", "i8", 1024, 2, 16), ("bf16", "fp8", 1671, 2, 16), ("bf16", "i8", 4096, 2, 8), ("bf16", "fp8", 4096, 4, 32), ("fp32", "fp8", 2048, 4, 8), ("fp32", "i8", 1003, 3, 16), ("bf16", "i8", 2051, 5, 8),
        ("bf16", "fp8", 8192, 2, 32)]


def rows_of(megabytes, beyond, dtype, K, N):
    return (megabytes << 20) // binding.slide_lifted_ld(K, N, dtype) + beyond


@pytest.mark.parametrize("act,dtype,K,N,last", ROWS)
@pytest.mark.parametrize("first", [True, False])
@pytest.mark.parametrize("beyond", [-1, 1])
def test_quantiser(act, dtype, K, N, last, first, beyond):
    M = rows_of(4 if first else last, beyond, dtype, K, N)
    gen = torch.Generator(device="cuda").manual_seed(K)
    X = torch.randn((M, K), generator=gen, device="cuda").to(torch.float32 if act == "fp32" else torch.bfloat16)
    q, s = binding.act_lift_quant(X, N, dtype)
    for rows in (slice(0, 5), slice(M // 2, M // 2 + 7), slice(M - 3, M)):
        qr, sr = binding.act_lift_quant(X[rows], N, dtype)
        assert torch.equal(q[rows].view(torch.uint8), qr.view(torch.uint8)) and (s is None or torch.equal(s[rows], sr))


@pytest.mark.parametrize("act,dtype,K,N", [("bf16", "i8", 4096, 4), ("bf16", "fp8", 2048, 2), ("bf16", "i8", 2048, 8), ("fp32", "i8", 2048, 3), ("bf16", "i8", 4104, 4)])
@pytest.mark.parametrize("beyond", [-1, 1])
def test_pruning(act, dtype, K, N, beyond):
    O = (4 << 20) // K + beyond
    gen = torch.Generator(device="cuda").manual_seed(K)
    W = torch.randn((O, K), generator=gen, device="cuda").to(torch.float32 if act == "fp32" else torch.bfloat16)
    Wq, s_w = binding.slide_prune_quant(W, N, dtype)
    for rows in (slice(0, 4), slice(O // 2, O // 2 + 4), slice(O - 3, O)):
        wr, sr = binding.slide_prune_quant(W[rows].contiguous(), N, dtype)
        assert torch.equal(Wq[rows].view(torch.uint8), wr.view(torch.uint8)) and torch.equal(s_w[rows], sr)
