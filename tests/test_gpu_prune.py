"""Offline weight path: the vector form of pruning + quantisation against the element-by-element one."""
import pytest
import torch

from paper_2603_05232_amd import binding

pytestmark = pytest.mark.gpu


# K: one unit, partial units, partial blocks, the longest rows held in registers and one vector more.  Moved by one
# element, the same matrix takes the element-by-element kernel, which defines the result, NaNs and infinities included.
@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("src", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("N,K", [(2, 16), (2, 16384), (2, 16392), (3, 24), (3, 104), (3, 24584), (4, 8), (4, 2056), (4, 18944), (4, 32776), (5, 40), (5, 5000),
                                 (5, 20488), (6, 24), (6, 1000), (7, 56), (7, 7168), (8, 16), (8, 1000)])
def test_prune_vector_form_matches_the_literal_one(dtype, src, N, K):
    O = 7
    gen = torch.Generator().manual_seed(K)
    W = (torch.randn((O, K), generator=gen) * 0.02).to(src)
    W[1] = (W[1] * 8).round() / 8                                     # mostly zeros and ties
    W[2] = torch.randint(-2, 3, (K,), generator=gen).to(src)
    W[3] = 0
    odd = torch.randperm(K, generator=gen)[: max(2, K // 50)]
    W[4, odd] = float("nan")
    W[5, odd[0]], W[5, odd[1]] = float("inf"), float("-inf")
    W[6] *= 1e-38                                                     # subnormal after the multiply
    flat = torch.zeros(O * K + 1, dtype=src, device="cuda")
    moved = flat[1:].view(O, K)
    moved.copy_(W.cuda())
    q1, s1 = binding.slide_prune_quant(W.cuda(), N, dtype)
    q2, s2 = binding.slide_prune_quant(moved, N, dtype)
    view = torch.int16 if q1.element_size() == 2 else torch.uint8
    assert torch.equal(q1.view(view), q2.view(view))
    if s1 is not None:
        assert torch.equal(s1.view(torch.int32), s2.view(torch.int32))
