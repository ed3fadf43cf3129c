"""The 256 x 256 tile kernel over lifted rows at the edges of its ring (rows of few units, and the shortest that go elsewhere), of
its tiles and of its rounds, against a product in 64 bits.  Operands are small integers, so every partial sum is exact in
all types."""
import pytest

from test_gpu_mid_tiles import _linear

pytestmark = pytest.mark.gpu


def _k(units, N, dtype):
    """A row length whose lifted row is `units` units of 128 bytes long, the last block cut short."""
    es = 1 if dtype in ("i8", "fp8") else 2
    blocks = max(1, 128 * units // es // (4 * (N - 1)))
    return blocks * 2 * N - 1


# 17 x 9 tiles: one partial round; the last tiles hold 52 tokens and 121 to 128 channels
@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16", "fp16"])
@pytest.mark.parametrize("units", [1, 2, 3, 4, 5, 6, 7, 8, 11])
def test_units(dtype, units):
    _linear(2100, 4224 - units, _k(units, 3 + units % 4, dtype), 3 + units % 4, dtype, False, False, units)


# more tiles than compute units (256): tiles that follow one another in a workgroup, with tokens and channels that end
# inside a tile
@pytest.mark.parametrize("dtype", ["i8", "fp8", "bf16"])
@pytest.mark.parametrize("M,O,units", [(4300, 4400, 3), (4300, 4400, 4), (4300, 4400, 5), (8100, 9000, 4), (8100, 9000, 7), (257, 66000, 6)])
def test_rounds(dtype, M, O, units):
    _linear(M, O, _k(units, 4, dtype), 4, dtype, False, False, units)
