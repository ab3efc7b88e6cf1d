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


def test_parts_in_turn_give_the_same_bits():
    """m2rnn_fwd_static with partial sums larger than its scratch: the parts of a state one after
    the other, against the side-by-side kernel on a full workspace."""
    import torch
    from paper_2603_14360_amd import binding as mb
    B, T, N, K, V = 1, 601, 16, 64, 64
    desc = mb.make_desc(B, T, N, K, V, mb.M2RNN_F32)
    need = mb.m2rnn_workspace_bytes(desc, 0)
    assert need > mb.M2RNN_STATIC_SCRATCH_BYTES
    print("case static fp32 forward", flush=True)
    inp = make_inputs(Workload("t", B, T, N, K, V, "f32", 9, K ** -0.5, 1.0, use_H0=True))
    dev = gu.to_device(inp, "f32")
    stream = torch.cuda.current_stream().cuda_stream
    w_r = torch.randn(N, V, device="cuda")
    outs = []
    for static in (False, True):
        y, HT = torch.full((B, T, N, V), float("nan"), device="cuda"), torch.empty(B, N, K, V, device="cuda")
        args = (dev["q"], dev["k"], dev["v"], dev["f"], dev["W"], dev["H0"], y, HT, None)
        if static:
            mb.m2rnn_fwd_static(desc, mb.make_opts(w_r=w_r), *args, stream=stream)
        else:
            ws = torch.empty(need, dtype=torch.uint8, device="cuda")
            mb.m2rnn_fwd_opt(desc, mb.make_opts(w_r=w_r), *args, ws, stream=stream)
        torch.cuda.synchronize()
        outs.append((y, HT))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
