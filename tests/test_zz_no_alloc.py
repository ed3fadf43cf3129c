"""slide_sparse_gemm_static (scratch in a static device array, nothing allocated) against slide_sparse_gemm_ws on the
same inputs: calls in a row, the later ones on smaller inputs, all bit for bit.  (Named to be collected last.)"""
import pytest
import torch

from paper_2603_05232_amd import binding, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# tokens, channels, elements per row: split rows on 15 tiles of 128 x 128, on fewer (the start of the same scratch array again), and of few tokens; then unsplit ones on small tiles
CASES = [(300, 640, 8192), (130, 384, 8192), (16, 3584, 18944)]
UNSPLIT = [(300, 640, 2048), (130, 384, 2048)]


def _case(M, O, K, N, seed):
    X = torch.from_numpy(synth.activations(M, K, seed=seed)).to(DEV)
    W = torch.from_numpy(synth.weights(O, K, seed=seed)).to(DEV)
    Wq, s_w = binding.slide_prune_quant(W, N, "i8")
    w_vals, w_meta = binding.slide_decompose(Wq, N, "i8")
    XL, s_x = binding.act_lift_quant(X, N, "i8")
    n = binding.slide_gemm_workspace_bytes(M, O, XL.shape[1], "i8")
    assert 0 < n <= binding.slide_static_scratch_bytes()
    ws = torch.full((n,), 0x5A, dtype=torch.uint8, device=DEV)
    Y_ws = binding.slide_sparse_gemm(XL, s_x, w_vals, w_meta, s_w, O, "i8", workspace=ws)
    Y_st = torch.full((M, O), -1.0, dtype=torch.bfloat16, device=DEV)
    binding.slide_sparse_gemm_static(XL, s_x, w_vals, w_meta, s_w, O, "i8", out=Y_st)
    torch.cuda.synchronize()
    assert torch.equal(Y_st.view(torch.int16), Y_ws.view(torch.int16))
    assert bool((ws != 0x5A).any()) == ((M, O, K) in CASES), "partial sums were written where the k range is split, and nowhere else"


def test_static_scratch_matches_workspace_call_twice():
    assert binding.slide_static_scratch_bytes() == 16 << 20
    for seed, (M, O, K) in enumerate(CASES + UNSPLIT):
        _case(M, O, K, 4, seed=seed + 1)


def test_static_scratch_rejects_bad_arguments():
    Y = torch.empty((4, 128), dtype=torch.bfloat16, device=DEV)
    x = torch.zeros((4, 100), dtype=torch.int8, device=DEV)
    s = torch.ones((128,), dtype=torch.float32, device=DEV)
    with pytest.raises(binding.SlideSparseError) as e:
        binding.slide_sparse_gemm_static(x, s[:4], x, x, s, 128, "i8", out=Y)      # K' not a multiple of 128
    assert e.value.code == 3
