"""GPU: a NaN in the scan reaches the outputs that depend on it and no other.  y_t depends on the
inputs of steps <= t; dq, dk, dv, df of step t on dy of steps >= t (and on the state, which is finite
here).  Inputs hold one NaN; every output that cannot depend on it keeps its bits."""
import pytest

from paper_2603_14360_amd import binding as mb
from paper_2603_14360_amd.synth_inputs import Workload, make_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu

T = 37
# (K, V, states): the splits of the 8-row forward, and its neighbours
FORWARD = [(64, 64, 2), (64, 64, 130), (128, 128, 2), (32, 32, 3), (32, 32, 300), (32, 32, 700), (16, 16, 3), (64, 16, 3),
           (64, 16, 140), (64, 32, 3), (64, 32, 150), (64, 32, 500), (32, 16, 3), (32, 16, 200), (64, 64, 600), (128, 32, 3)]


def _device(K, V, units, io):
    wl = Workload("t", units, T, 1, K, V, io, 50 + K + V, K ** -0.5, 1.0, use_H0=True, use_dHT=True)
    return gu.to_device(make_inputs(wl), io)


@pytest.mark.parametrize("io,K,V,units", [("bf16",) + c for c in FORWARD] +
                         [("f32", K, V, 2) for K in (16, 64) for V in (16, 32, 64)])
@pytest.mark.parametrize("t", [5, 21])
def test_y_of_earlier_steps(io, K, V, units, t):
    import torch
    print("case", io, K, V, units, t, flush=True)
    dev = _device(K, V, units, io)
    scan = mb.Scan(units, T, 1, K, V, io, backward=False)
    args = lambda: (dev["q"], dev["k"], dev["v"], dev["f"], dev["W"], dev["H0"])
    clean, H = (x.clone() for x in scan.fwd(*args()))
    dev["v"][0, t, 0, 3] = float("nan")
    y, HT = scan.fwd(*args())
    torch.cuda.synchronize()
    assert torch.equal(y[0, :t], clean[0, :t])
    assert torch.equal(y[1:], clean[1:]) and torch.equal(HT[1:], H[1:])
    assert y[0, t:, 0, 3].isnan().all() and y[0, t + 1:].isnan().all() and HT[0].isnan().all()


# the backwards in fp32 throughout, V <= 64 and V = 128 (fp32 io, and bf16 io of the shapes without
# a matrix-core backward)
FP32_BACKWARD = [("f32", K, V) for K in (16, 64) for V in (16, 32, 64)] + [("f32", 32, 128)]
FP32_BACKWARD += [("bf16", 64, 32), ("bf16", 128, 64), ("bf16", 16, 64)]


@pytest.mark.parametrize("io,K,V", FP32_BACKWARD)
@pytest.mark.parametrize("t,bad", [(5, "nan"), (21, "nan"), (21, "inf")])
def test_gradients_of_later_steps(io, K, V, t, bad):
    """dy of step t holds one NaN or infinity: the gradients of the steps behind t, which do not
    depend on it, keep their bits; those of the steps up to t are spoiled."""
    import torch
    units = 2
    print("case", io, K, V, t, bad, flush=True)
    dev = _device(K, V, units, io)
    scan = mb.Scan(units, T, 1, K, V, io)
    args = [dev[n] for n in ("q", "k", "v", "f", "W", "H0")]
    scan.fwd(*args)
    grads = lambda: [x.clone() for x in scan.bwd(*args, dev["dy"], dev["dHT"])]
    clean = grads()
    dev["dy"][0, t, 0, 3] = float(bad)
    got = grads()
    torch.cuda.synchronize()
    for name, g, c in zip(gu.GRAD_NAMES[:4], got, clean):
        assert torch.equal(g[0, t + 1:], c[0, t + 1:]), name
        assert torch.equal(g[1:], c[1:]), name
    dq, dk, dv, df = got[:4]
    assert not df[0, :t + 1].isfinite().any() and not dv[0, :t, 0].isfinite().any()
    assert torch.equal(got[5][1:], clean[5][1:]) and not got[4].isfinite().any()


@pytest.mark.parametrize("K,V,units", [(64, 64, 2), (64, 64, 130), (128, 128, 2), (32, 32, 3), (32, 32, 600), (16, 16, 3),
                                       (32, 16, 3), (64, 16, 3), (64, 16, 300), (128, 16, 2)])
@pytest.mark.parametrize("t", [5, 21, 36])
def test_df_of_later_steps_in_the_matrix_core_backwards(K, V, units, t):
    """dy of step t holds one NaN: df of the steps behind t keeps its bits, also within a chunk.  (dq, dk and
    dv of a chunk are products that hold all its steps side by side, zeros in the places of the others.)"""
    import torch
    print("case df", K, V, units, t, flush=True)
    dev = _device(K, V, units, "bf16")
    scan = mb.Scan(units, T, 1, K, V, "bf16")
    args = [dev[n] for n in ("q", "k", "v", "f", "W", "H0")]
    scan.fwd(*args)
    grads = lambda: [x.clone() for x in scan.bwd(*args, dev["dy"], dev["dHT"])]
    clean = grads()
    small = dev["dy"][0, t, 0].abs().argmin()   # (the largest entries set the scale of a chunk)
    dev["dy"][0, t, 0, small] = float("nan")
    got = grads()
    torch.cuda.synchronize()
    assert torch.equal(got[3][0, t + 1:], clean[3][0, t + 1:])
    assert not got[3][0, :t + 1].isfinite().any()
    for name, g, c in zip(gu.GRAD_NAMES, got, clean):
        assert name == "dW" or torch.equal(g[1:], c[1:]), name
