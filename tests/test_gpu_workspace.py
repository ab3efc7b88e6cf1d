"""GPU: calls on exactly the workspace they ask for, bytes behind it guarded; the backward that
recomputes its checkpoints; a NULL workspace with a size beside it."""
import ctypes

import pytest

from paper_2603_14360_amd import binding as mb
from paper_2603_14360_amd.synth_inputs import Workload, make_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu

SHAPES = [(64, 64, 3), (64, 64, 40), (128, 128, 2), (128, 128, 20), (32, 32, 3), (16, 16, 3), (64, 16, 5), (64, 32, 5),
          (32, 16, 3), (128, 64, 2), (64, 128, 2)]


def _guarded(nbytes):
    import torch
    buf = torch.full((nbytes + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    return buf, buf[:nbytes]


@pytest.mark.parametrize("io", ["bf16", "f32"])
@pytest.mark.parametrize("K,V,units", SHAPES)
def test_exact_sizes_and_recomputed_checkpoints(io, K, V, units):
    import torch
    T = 53
    print("case", io, K, V, units, flush=True)
    dev = gu.to_device(make_inputs(Workload("t", units, T, 1, K, V, io, 5, K ** -0.5, 1.0, use_H0=True, use_dHT=True)), io)
    scan = mb.Scan(units, T, 1, K, V, io)
    args = [dev[n] for n in ("q", "k", "v", "f", "W", "H0")]
    st = torch.cuda.current_stream().cuda_stream
    outs = []
    for use_ckpt in (True, False):
        for t in (scan.y, scan.HT, scan.dq, scan.dk, scan.dv, scan.df, scan.dW, scan.dH0):
            t.fill_(float("nan"))
        buf, ws = _guarded(mb.m2rnn_workspace_bytes(scan.desc, 0))
        mb.m2rnn_fwd(scan.desc, *args, scan.y, scan.HT, scan.ckpt, ws, stream=st)
        buf2, ws2 = _guarded(mb.m2rnn_workspace_bytes(scan.desc, 1 if use_ckpt else 2))
        mb.m2rnn_bwd(scan.desc, *args, scan.ckpt if use_ckpt else None, dev["dy"], dev["dHT"], scan.dq, scan.dk, scan.dv,
                     scan.df, scan.dW, scan.dH0, ws2, stream=st)
        torch.cuda.synchronize()
        assert (buf[ws.numel():] == 0xFF).all() and (buf2[ws2.numel():] == 0xFF).all()
        outs.append([t.clone() for t in (scan.y, scan.HT, scan.dq, scan.dk, scan.dv, scan.df, scan.dW, scan.dH0)])
    for x, y in zip(*outs):
        assert torch.isfinite(x.float()).all() and torch.equal(x, y)


@pytest.mark.parametrize("K,V,units", [(64, 32, 4), (32, 16, 3), (32, 32, 300), (16, 16, 40)])
def test_null_workspace_with_a_size(K, V, units):
    import torch
    T = 37
    print("case null workspace", K, V, units, flush=True)
    dev = gu.to_device(make_inputs(Workload("t", units, T, 1, K, V, "bf16", 5, K ** -0.5, 1.0, use_H0=True)), "bf16")
    desc = mb.make_desc(units, T, 1, K, V, mb.M2RNN_BF16)
    scan = mb.Scan(units, T, 1, K, V, "bf16", backward=False)
    args = [dev[n] for n in ("q", "k", "v", "f", "W", "H0")]
    y, HT = (x.clone() for x in scan.fwd(*args))
    y2, HT2 = torch.full_like(y, float("nan")), torch.full_like(HT, float("nan"))
    p = lambda x: ctypes.c_void_p(x.data_ptr())
    rc = mb.lib().m2rnn_fwd(ctypes.byref(desc), *map(p, args), p(y2), p(HT2), None, None, 1 << 30,
                            ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0 and torch.equal(y, y2) and torch.equal(HT, HT2)
