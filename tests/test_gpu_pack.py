"""Offline weight path: the packed layout word by word against the oracle's decomposition."""
import numpy as np
import pytest
import torch

from oracle import slide_oracle as so
from paper_2603_05232_amd import binding, synth
from test_gpu_parity import dev, host, to_dev_q

pytestmark = pytest.mark.gpu
PANEL = 128


def expected_packed(Wq, N, dtype, fused):
    """The layout of packed_layout.h written out with numpy from the canonical windows."""
    es = 1 if dtype in ("i8", "fp8") else 2
    ev, ei = so.compress_24(so.slide_decompose(Wq, N, dtype), dtype)
    O, K = Wq.shape
    nwin, nw, hw, bl = ei.shape[1], 8 // es, 4 // es, 8 // es          # windows of a row; per lane; per lane and step half; blocks per half line
    nsteps = 3 * (-(-K * es // 128)) if fused else binding.slide_lifted_ld(K, N, dtype) * es // 64
    npanels = -(-O // PANEL)
    j = np.empty((nsteps, 2, nw), dtype=np.int64)
    for s in range(nsteps):
        for qa in range(2):
            for w in range(nw):
                if fused:
                    qb, wsl, J = w // hw, hw * qa + w % hw, s % 3
                    g = (2 * (s // 3) + qb) * bl + (wsl if J == 2 else J * (bl // 2) + (wsl >> 1))
                    j[s, qa, w] = g * 3 + (1 if J == 2 else 2 * (wsl & 1))
                else:
                    j[s, qa, w] = s * 2 * nw + 2 * hw * (w // hw) + hw * qa + w % hw
    exists = j < nwin
    jc = np.where(exists, j, 0)
    vals = np.zeros((npanels, nsteps, 4, 64, 2 * nw), dtype=ev.dtype)
    meta = np.zeros((npanels, nsteps, 64, 4), dtype=np.uint32)
    shifts = 4 * np.arange(nw)
    for p in range(npanels):
        for f in range(4):
            for lane in range(64):
                i, qa = lane & 31, lane >> 5
                o = p * PANEL + 64 * ((i >> 2) & 1) + 16 * f + 4 * (i >> 3) + (i & 3)
                win = jc[:, qa]
                here = exists[:, qa] & (o < O)
                row = min(o, O - 1)
                pair = ev[row].reshape(nwin, 2)[win]
                vals[p, :, f, lane] = np.where(here[..., None], pair, 0).reshape(nsteps, 2 * nw)
                pos = np.where(here, ei[row][win], 4).astype(np.uint32)
                meta[p, :, lane, f] = (pos << shifts).sum(axis=1).astype(np.uint32)
    return vals, meta


def _placed(a, offset, dtype):
    """A contiguous device matrix whose first element lies `offset` elements into its allocation."""
    flat = torch.zeros(a.size + offset, dtype=to_dev_q(a[:1, :1], dtype).dtype, device="cuda")
    t = flat[offset:].view(a.shape)
    t.copy_(to_dev_q(a, dtype))
    return t


# whole and partial groups of 16 / ES blocks, partial panels, rows of any length, matrices that start off a 16-byte line
@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("N,O,K,offset,fused", [(4, 130, 512, 0, True), (4, 96, 136, 0, True), (4, 33, 1000, 0, True), (4, 17, 77, 3, True), (4, 9, 64, 1, True),
                                                (2, 33, 320, 0, False), (3, 129, 96, 0, False), (3, 20, 101, 0, False), (4, 40, 384, 0, False),
                                                (4, 40, 384, 1, False), (5, 31, 333, 5, False), (5, 7, 3, 0, False), (6, 18, 432, 0, False),
                                                (7, 12, 450, 2, False), (8, 16, 528, 0, False), (8, 5, 17, 1, False)])
def test_packed_layout_matches_the_oracle(dtype, N, O, K, offset, fused):
    Wq, _ = so.prepare_weights(synth.weights(O, K, seed=N + K), N, dtype)
    Wq = Wq.copy()
    rng = np.random.default_rng(K)
    Wq[rng.random(Wq.shape) < 0.25] = 0
    if dtype != "i8":
        Wq[rng.random(Wq.shape) < 0.1] = 0x80 if dtype == "fp8" else 0x8000          # -0 is no non-zero and is never stored
    ev, em = expected_packed(Wq, N, dtype, fused)
    pack = binding.slide_decompose_fused if fused else binding.slide_decompose
    gv, gm, viol = pack(_placed(Wq, offset, dtype), N, dtype, count_violations=True)
    assert int(host(viol)[0]) == 0
    assert np.array_equal(host(gm).view(np.uint32), em.reshape(-1))
    assert np.array_equal(host(gv).view(np.uint8), ev.reshape(-1).view(np.uint8))
