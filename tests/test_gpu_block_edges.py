"""GPU parity of the block kernels at the edges of their launches: feature counts around whole
waves, token counts around the rows of the ordered sums (one launch or two) and beyond the
workgroups that walk them."""
import pytest

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
