"""GPU parity for EVERY scan kernel that the library compiles: each split of the 8-row forward, each
tiling and each one-wave-per-row-block shape, the fp32 kernels, decode, with and without gradient
clipping and the forward's checkpoints, against the float64 oracle, with B*N and T chosen so that the
call is really routed to the variant named in the test id (m2rnn_route_string tells which one serves a
descriptor).  H0 and dH_T set.  tests/test_dispatch_cpu.py holds this file to its claim: it records
what these cases launch and compares that with the kernels in the library."""
import pytest

from paper_2603_14360_amd import binding as mb
from paper_2603_14360_amd.synth_inputs import Workload, make_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu

# (K, V, B, N, Nqk, forward route, backward route), bf16, T = 35
CASES = [
    # 8-row forward, matrix-core backward tilings
    (64, 64, 8, 16, 0, "half<64,64,4>", "tile<64,64,2>"),
    (64, 64, 10, 4, 0, "half<64,64,2>", "tile<64,64,1>"),
    (64, 64, 3, 5, 0, "half<64,64,1>", "tile<64,64,1>"),
    (128, 128, 2, 3, 0, "half<128,128,1>", "tile<128,128,1>"),
    (32, 32, 16, 16, 0, "half<32,32,4>", "tile<32,32,2>"),
    (32, 32, 16, 24, 4, "half<32,32,4>", "tile<32,32,2>"),
    (32, 32, 3, 5, 0, "half<32,32,4>", "tile<32,32,1>"),
    (16, 16, 3, 5, 0, "half<16,16,2>", "rowwave_bwd<16,16>"),
    (64, 16, 3, 5, 0, "half<64,16,8>", "rowwave_bwd<64,16>"),
    (64, 32, 2, 3, 0, "half<64,32,1>", "quad<64,32>"),
    (32, 16, 2, 3, 0, "half<32,16,4>", "rowwave_bwd<32,16>"),
    # 16-row forward
    (128, 128, 5, 4, 0, "tile<128,128,1>", "tile<128,128,1>"),
    (32, 32, 27, 20, 0, "tile<32,32,2>", "tile<32,32,2>"),
    # one wave per row block (forward), paired with a matrix-core backward ...
    (64, 64, 32, 16, 0, "rowwave<64,64>", "tile<64,64,2>"),
    (32, 32, 32, 32, 0, "rowwave<32,32>", "tile<32,32,2>"),
    (16, 16, 32, 64, 0, "rowwave<16,16>", "rowwave_bwd<16,16>"),
    (64, 16, 8, 84, 1, "rowwave<64,16>", "rowwave_bwd<64,16>"),
    (32, 16, 32, 32, 8, "rowwave<32,16>", "rowwave_bwd<32,16>"),
    (128, 16, 2, 3, 0, "rowwave<128,16>", "rowwave_bwd<128,16>"),
    # ... or with the fp32 backward where no matrix-core backward exists
    (16, 32, 2, 3, 0, "rowwave<16,32>", "quad<16,32>"),
    (64, 32, 32, 16, 0, "rowwave<64,32>", "quad<64,32>"),
    (128, 32, 2, 3, 0, "rowwave<128,32>", "quad<128,32>"),
    (16, 64, 2, 3, 0, "rowwave<16,64>", "quad<16,64>"),
    (32, 64, 2, 3, 0, "rowwave<32,64>", "quad<32,64>"),
    (128, 64, 2, 3, 0, "rowwave<128,64>", "quad<128,64>"),
    # shapes with V = 128 and K != V: vector-ALU kernels both ways
    (16, 128, 1, 2, 0, "generic<bf16>", "generic<bf16>"),
    (64, 128, 1, 2, 0, "generic<bf16>", "generic<bf16>"),
]
# splits of the 8-row forward that other state counts and longer sequences take: (K, V, B, N, T, route)
SPLITS = [
    (32, 32, 3, 5, 261, "half<32,32,1>"), (32, 32, 20, 5, 261, "half<32,32,2>"),
    (16, 16, 3, 5, 261, "half<16,16,1>"), (64, 16, 3, 5, 261, "half<64,16,1>"),
    (64, 16, 10, 4, 261, "half<64,16,2>"), (64, 16, 10, 8, 261, "half<64,16,4>"),
    (32, 16, 3, 5, 261, "half<32,16,1>"), (32, 16, 10, 8, 261, "half<32,16,2>"),
    (64, 32, 10, 4, 35, "half<64,32,2>"), (64, 32, 10, 9, 35, "half<64,32,4>"), (64, 32, 10, 21, 35, "half<64,32,8>"),
    (32, 32, 20, 13, 261, "half<32,32,2>"), (64, 32, 10, 13, 261, "half<64,32,2>"), (64, 32, 10, 13, 35, "half<64,32,8>"),
    (64, 64, 10, 7, 35, "half<64,64,1>"),
]
# ... and that the checkpoint pass of the backward takes: (K, V, states)
CHECKPOINT_PASS = [(16, 16, 200), (32, 16, 100), (32, 16, 300), (64, 16, 40), (64, 16, 100), (64, 16, 200), (64, 32, 40),
                   (64, 32, 90), (64, 32, 210), (32, 32, 5), (32, 32, 100), (32, 32, 300), (64, 64, 40), (64, 64, 120),
                   (64, 32, 130), (64, 64, 4), (64, 64, 70), (64, 32, 4)]
DECODE = [(K, V) for V in (16, 32, 64) for K in (16, 32, 64, 128)]
# V = 128 in fp32 on the vector ALUs, W beside the state in LDS (forward, backward) or not
GENERIC_F32 = [(16, 128), (64, 128), (128, 128)]


@pytest.mark.parametrize("K,V,B,N,Nqk,fwd_route,bwd_route", CASES,
                         ids=["%s+%s@K%dV%dB%dN%d" % (c[5], c[6], c[0], c[1], c[2], c[3]) for c in CASES])
def test_every_dispatch_route(K, V, B, N, Nqk, fwd_route, bwd_route):
    T = 35
    desc = mb.make_desc(B, T, N, K, V, mb.M2RNN_BF16, Nqk=(Nqk or None))
    assert mb.m2rnn_route_string(desc, 0) == fwd_route
    assert mb.m2rnn_route_string(desc, 1) == bwd_route
    label = "route %s / %s" % (fwd_route, bwd_route)
    print("case", label, "B%d N%d" % (B, N), flush=True)
    wl = Workload("t", B, T, N, K, V, "bf16", 900 + K + 3 * V + B, K ** -0.5, 1.0, use_H0=True,
                  use_dHT=True, Nqk=Nqk)
    inp = make_inputs(wl)
    got = gu.run_gpu(inp, "bf16")
    ref = gu.run_oracle(inp)
    errs = gu.compare(got, ref, gu.TOL["bf16"], label=label)
    print(label, {k: float("%.3g" % v) for k, v in errs.items()}, flush=True)
    # the backward that recomputes the checkpoints (forward kernels without the readout): same bits
    again = gu.run_gpu(inp, "bf16", use_ckpt=False)
    assert all((again[n] == got[n]).all() for n in got)


# (one case of every backward kernel)
CLIPPED = sorted({c[6]: c for c in CASES}.values())


@pytest.mark.parametrize("K,V,B,N,Nqk,fwd_route,bwd_route", CLIPPED, ids=[c[6] + "@K%dV%d" % c[:2] for c in CLIPPED])
def test_every_backward_with_clipping(K, V, B, N, Nqk, fwd_route, bwd_route):
    print("case clipped", bwd_route, K, V, flush=True)
    inp = make_inputs(Workload("t", B, 35, N, K, V, "bf16", 950 + K + 3 * V + B, K ** -0.5, 1.0, use_H0=True,
                               use_dHT=True, Nqk=Nqk))
    gu.compare(gu.run_gpu(inp, "bf16", grad_clip=0.5), gu.run_oracle(inp, grad_clip=0.5), gu.TOL["bf16"], label=bwd_route)


@pytest.mark.parametrize("K,V,B,N,T,route", SPLITS, ids=["%s-B%dN%d" % (c[5], c[2], c[3]) for c in SPLITS])
def test_splits_of_the_8_row_forward(K, V, B, N, T, route):
    assert mb.m2rnn_route_string(mb.make_desc(B, T, N, K, V, mb.M2RNN_BF16), 0) == route
    print("case", route, flush=True)
    inp = make_inputs(Workload("t", B, T, N, K, V, "bf16", 800 + K + 3 * V + B, K ** -0.5, 1.0, use_H0=True))
    gu.compare(gu.run_gpu(inp, "bf16", backward=False), gu.run_oracle(inp, backward=False), gu.TOL["bf16"], label=route)


@pytest.mark.parametrize("K,V,units", CHECKPOINT_PASS)
def test_splits_of_the_checkpoint_pass(K, V, units):
    print("case checkpoint pass", K, V, units, flush=True)
    inp = make_inputs(Workload("t", units, 35, 1, K, V, "bf16", 850 + K + 3 * V, K ** -0.5, 1.0, use_H0=True, use_dHT=True))
    got, again = gu.run_gpu(inp, "bf16"), gu.run_gpu(inp, "bf16", use_ckpt=False)
    assert all((again[n] == got[n]).all() for n in got)


@pytest.mark.parametrize("K,V", DECODE)
def test_decode_shapes(K, V):
    assert mb.m2rnn_route_string(mb.make_desc(5, 1, 3, K, V, mb.M2RNN_BF16), 0) == "decode<%d,%d>" % (K, V)
    print("case decode", K, V, flush=True)
    inp = make_inputs(Workload("t", 5, 1, 3, K, V, "bf16", 700 + K + 3 * V, K ** -0.5, 1.0, use_H0=True))
    gu.compare(gu.run_gpu(inp, "bf16", backward=False), gu.run_oracle(inp, backward=False), gu.TOL["bf16"], label="decode")


@pytest.mark.parametrize("K,V", GENERIC_F32)
def test_generic_f32(K, V):
    assert mb.m2rnn_route_string(mb.make_desc(2, 35, 3, K, V, mb.M2RNN_F32), 0) == "generic<f32>"
    print("case generic f32", K, V, flush=True)
    inp = make_inputs(Workload("t", 2, 35, 3, K, V, "f32", 600 + K, K ** -0.5, 1.0, use_H0=True, use_dHT=True))
    gu.compare(gu.run_gpu(inp, "f32"), gu.run_oracle(inp), gu.TOL["f32"], label="generic f32")
