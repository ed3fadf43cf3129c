"""The two encoders of the quantisers (conversion instruction / rounding by addition, and the literal one) on every value
where they could part: all codes, the midpoints between neighbours and the floats either side of each midpoint."""
import numpy as np
import pytest
import torch

from oracle import slide_oracle as so
from paper_2603_05232_amd import binding

pytestmark = pytest.mark.gpu


def _values(dtype):
    """Positive values, ending with the full scale (so that a row that holds them all is quantised with factor 1)."""
    if dtype == "fp8":
        grid = np.unique(np.abs(so.fp8_e4m3_decode(np.arange(0x7F, dtype=np.uint8)))).astype(np.float32)      # 0 .. 448
    else:
        grid = np.arange(128, dtype=np.float32)
    mid = ((grid[1:].astype(np.float64) + grid[:-1]) / 2).astype(np.float32)                                    # exact
    inf = np.float32(np.inf)
    v = np.concatenate([grid, mid, np.nextafter(mid, inf), np.nextafter(mid, -inf), np.nextafter(grid[1:], -inf)])
    return np.concatenate([v, [np.float32(1e-40), grid[-1]]]).astype(np.float32)


def _expected(v, dtype):
    return so.fp8_e4m3_encode(v) if dtype == "fp8" else np.rint(v).astype(np.int8)


@pytest.mark.parametrize("dtype", ["i8", "fp8"])
@pytest.mark.parametrize("tail", [0, 1])                        # whole 16-byte vectors; element by element
def test_activations(dtype, tail):
    v = _values(dtype)
    K = (v.size + 15) // 16 * 16 + tail
    X = np.zeros((2, K), dtype=np.float32)
    X[0, : v.size], X[1, : v.size] = v, -v
    for N in (2, 4):
        XL, s = binding.act_lift_quant(torch.from_numpy(X).cuda(), N, dtype)
        exp = so.lift(_expected(X, dtype), N)
        assert np.array_equal(s.cpu().numpy(), np.ones(2, dtype=np.float32))
        assert np.array_equal(XL.cpu().numpy()[:, : exp.shape[1]], exp)


@pytest.mark.parametrize("dtype", ["i8", "fp8"])
@pytest.mark.parametrize("offset", [0, 1])                      # vector form; moved by one element, element by element
def test_weights(dtype, offset):
    v = _values(dtype)
    v = np.concatenate([v, np.zeros(v.size % 2, dtype=np.float32)])
    W = np.zeros((2, v.size * 2), dtype=np.float32)             # two values and two zeros to a block of 2:4: nothing is pruned
    W[0, 0::4], W[0, 1::4] = v[0::2], v[1::2]
    W[1] = -W[0]
    flat = torch.zeros(W.size + offset, dtype=torch.float32, device="cuda")
    t = flat[offset:].view(W.shape)
    t.copy_(torch.from_numpy(W))
    Wq, s = binding.slide_prune_quant(t, 2, dtype)
    exp = _expected(W, dtype)
    got = Wq.cpu().numpy()
    if dtype == "fp8":                                          # pruned zeros are +0; a kept -0 keeps its sign
        exp, got = np.where(exp == 0x80, 0, exp), np.where(got == 0x80, 0, got)
    assert np.array_equal(s.cpu().numpy(), np.ones(2, dtype=np.float32))
    assert np.array_equal(got, exp)
