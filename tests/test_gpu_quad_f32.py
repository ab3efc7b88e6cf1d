"""The fp32 kernels on the 4x4x1 matrix instructions (V <= 64): every shape they are compiled for,
at lengths around the 16-step blocks, and with checkpoint intervals below, at and above the 16
steps that the backward keeps on chip (above: it re-runs a chunk once to place inner states).
fp32 io, 1e-5 as everywhere: two roundings of 6e-8 per step over at most 50 steps of a recurrence
whose gain is about one stay below 1e-5 of the largest entry."""
import pytest

from paper_2603_14360_amd.synth_inputs import Workload, make_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu

SHAPES = [(K, V) for V in (16, 32, 64) for K in (16, 32, 64, 128)]


def _check(B, T, N, K, V, chunk, Nqk=0, clip=0.0, io="f32"):
    label = "quad K%d V%d T%d C%d Nqk%d" % (K, V, T, chunk, Nqk)
    print("case", label, flush=True)
    wl = Workload("t", B, T, N, K, V, io, 70 + K + V + T, K ** -0.5, 1.0, use_H0=True, use_dHT=True, Nqk=Nqk)
    inp = make_inputs(wl)
    got = gu.run_gpu(inp, io, chunk=chunk, grad_clip=clip)
    gu.compare(got, gu.run_oracle(inp, grad_clip=clip), gu.TOL[io], label=label)


@pytest.mark.parametrize("K,V", SHAPES)
def test_shapes(K, V):
    _check(2, 35, 3, K, V, 0)


@pytest.mark.parametrize("T,chunk", [(1, 0), (15, 0), (16, 0), (17, 0), (33, 5), (33, 16), (50, 17), (50, 33), (49, 256)])
@pytest.mark.parametrize("K,V", [(32, 32), (64, 16), (64, 64)])
def test_lengths_and_intervals(K, V, T, chunk):
    _check(1, T, 4, K, V, chunk, Nqk=2, clip=0.5 if T == 33 else 0.0)
