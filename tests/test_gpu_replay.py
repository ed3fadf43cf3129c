"""Every route of the sparse GEMMs that has a kernel or a launch of its own, captured into a HIP graph and on a stream other than
the default one: each result bit by bit that of a call on the default stream (which the tests of these kernels compare with a
product in 64 bits)."""
import pytest
import torch

from paper_2603_05232_amd import binding

pytestmark = pytest.mark.gpu

# name: fused, tokens, channels, elements per row, workspace
ROUTES = {"narrow tiles": (True, 1100, 4224, 640, False),
          "large tiles and a rest on narrow ones": (True, 2048, 32 * 256 + 3142, 2048, False),
          "large tiles in rounds, odd rows": (True, 8100, 9000, 384, False),
          "large tiles in rounds, even rows": (True, 8100, 9000, 512, False),
          "five fragments a workgroup": (True, 17, 257 * 128, 2048, False),
          "stream of a panel": (True, 17, 192 * 128, 1152, False),
          "stream of a panel, split rows": (True, 9, 300, 16768, True),
          "two groups of wavefronts": (False, 17, 130 * 128, 1536, False),
          "lifted tiles in rounds": (False, 8100, 9000, 411, False),
          "lifted tiles in rounds, short rows": (False, 8100, 9000, 160, False),
          "lifted tiles, one round": (False, 2100, 4224, 1003, False),
          "sixteen channels a workgroup, unlifted": (True, 9, 1000, 2048, True),
          "sixteen channels a workgroup, lifted": (False, 16, 4096, 1003, False),
          "small tiles, 1 x 1": (True, 40, 700, 2176, True),
          "small tiles, 2 x 2": (False, 250, 4096, 2560, True),
          "small tiles, 2 x 3": (True, 256, 42 * 128, 3584, True),
          "small tiles, 2 x 4": (False, 400, 30 * 128 - 5, 1003, False),
          "few-token kernel, unlifted": (True, 5, 65 * 128, 1408, False),
          "few-token kernel, lifted": (False, 15, 190 * 128 - 3, 600, False),
          "split tiles of 64 tokens": (True, 40, 600, 6656, True),
          "split tiles of 128 tokens": (False, 150, 700, 5632, True)}


@pytest.mark.parametrize("name", ROUTES)
def test_graph_replay_and_streams(name):
    fused, M, O, K, with_ws = ROUTES[name]
    gen = torch.Generator(device="cuda").manual_seed(M)
    xs = [torch.randn((M, K), generator=gen, device="cuda") for _ in range(3)]
    Wq, s_w = binding.slide_prune_quant(torch.randn((O, K), generator=gen, device="cuda"), 4, "i8")
    wv, wm = (binding.slide_decompose_fused if fused else binding.slide_decompose)(Wq, 4, "i8")
    row = K if fused else binding.slide_lifted_ld(K, 4, "i8")
    ws = torch.empty((binding.slide_gemm_workspace_bytes(M, O, row, "i8"),), dtype=torch.uint8, device="cuda") if with_ws else None
    assert "split" not in name or ws.numel() > 0

    def layer(x, q=None, s=None, y=None):
        q, s = binding.act_lift_quant(x, 2 if fused else 4, "i8", out=q, s_x=s)
        if fused:
            return binding.slide_sparse_gemm_fused(q, s, wv, wm, s_w, O, K, 4, "i8", out=y, workspace=ws)
        return binding.slide_sparse_gemm(q, s, wv, wm, s_w, O, "i8", out=y, workspace=ws)

    if ws is not None:
        ws.fill_(0x5A)
    refs = [layer(x) for x in xs]
    assert (ws is not None and bool((ws != 0x5A).any())) == ("split" in name)            # partial sums were written
    x_in, q = xs[0].clone(), torch.empty((M, row), dtype=torch.int8, device="cuda")
    s, y = torch.empty((M,), device="cuda"), torch.empty((M, O), dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        layer(x_in, q, s, y)
    for i in (1, 2, 0, 1):
        x_in.copy_(xs[i])
        y.fill_(7.0)
        g.replay()
        assert torch.equal(y.view(torch.int16), refs[i].view(torch.int16)), f"replay with input {i}"
        assert torch.equal(layer(xs[2]), refs[2])                    # eager work between the replays
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = [layer(x) for x in xs]
    torch.cuda.current_stream().wait_stream(side)
    for a, b in zip(got, refs):
        a.record_stream(torch.cuda.current_stream())
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
