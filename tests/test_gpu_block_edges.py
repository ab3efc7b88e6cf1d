"""GPU parity of the block kernels at the edges of their launches: feature counts around whole
waves, token counts around the rows of the ordered sums (one launch or two) and beyond the
workgroups that walk them."""
import pytest

from test_gpu_block import test_conv_silu as conv_case
from test_gpu_block import test_gated_rmsnorm as norm_case

pytestmark = pytest.mark.gpu

# D: one lane, around one, two, three, five and six waves, the largest
NORM = [(1, 3, D, 1e-5, D % 16 == 0) for D in (8, 504, 512, 520, 1032, 1536, 1544, 2056, 3072, 3080, 4096)]
# tokens: around the direct sum's 512 rows, more than the workgroups of one or three waves
NORM += [(1, 512, 16, 1e-5, True), (1, 513, 16, 0.0, False), (3, 1500, 24, 1e-5, True), (2, 700, 1344, 1e-5, False)]


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,T,D,eps,cache", NORM)
def test_norm_edges(io, B, T, D, eps, cache):
    norm_case(io, B, T, D, eps, cache)


# C: one vector of channels, around a workgroup's 128, widths that divide it unevenly;
# T: around the shortest segment of 8 steps and its halo of 3
CONV = [(1, T, C, C % 16 == 0) for T in (5, 7, 8, 9, 11, 12, 17) for C in (8, 136)]
CONV += [(2, 61, C, True) for C in (120, 128, 264, 1016)] + [(300, 3, 24, True), (5, 1111, 264, False)]


@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,T,C,bias", CONV)
def test_conv_edges(io, B, T, C, bias):
    conv_case(io, B, T, C, bias)


# the longer segments, taken by launches that fill the chip: 16, 32 and 64 steps, ragged ends
@pytest.mark.parametrize("B,T,C,bias", [(3, 1399, 4000, True), (3, 2799, 4000, False), (17, 3901, 1024, True)])
def test_conv_long_segments(B, T, C, bias):
    conv_case("bf16", B, T, C, bias)
