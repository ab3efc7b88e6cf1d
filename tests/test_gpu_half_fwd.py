"""GPU parity of the forward on 8-row blocks: every split it is compiled for, T around its
16-step blocks, with and without options, and the promise that y has the same bits on every
split of a state (what a workspace has room for decides between splits)."""
import pytest

from paper_2603_14360_amd import binding as mb
from paper_2603_14360_amd.synth_inputs import Workload, make_inputs
import gpu_util as gu

pytestmark = pytest.mark.gpu

# state counts at which the launch rule turns from one split to the next
SHAPES = [(64, 64, (1, 32, 33, 65, 130)), (128, 128, (1, 16, 17)), (32, 32, (1, 65, 300, 513, 1000)),
          (16, 16, (1, 130)), (64, 16, (1, 70, 140)), (64, 32, (1, 40, 70, 150, 257, 385)), (32, 16, (3, 100, 200))]
CASES = [(K, V, n) for K, V, counts in SHAPES for n in counts]


@pytest.mark.parametrize("K,V,units", CASES, ids=["K%dV%d-%d" % c for c in CASES])
@pytest.mark.parametrize("T", [2, 16, 37])
def test_splits_against_oracle(K, V, units, T):
    print("case", K, V, units, T, flush=True)
    wl = Workload("t", units, T, 1, K, V, "bf16", 77 + K + V + T, K ** -0.5, 1.0, use_H0=True)
    inp = make_inputs(wl)
    dev = gu.to_device(inp, "bf16")
    scan = mb.Scan(units, T, 1, K, V, "bf16", backward=False)
    y, HT = scan.fwd(dev["q"], dev["k"], dev["v"], dev["f"], dev["W"], dev["H0"])
    ref = gu.run_oracle(inp, backward=False)
    errs = {"y": gu.rel_err(gu.to_np(y), ref["y"]), "HT": gu.rel_err(gu.to_np(HT), ref["HT"])}
    # y is a bf16 tensor: half an ulp, 2^-9; HT is fp32 from ~21-bit operands, T steps of 1e-8 each
    assert errs["y"] <= 2 ** -8 and errs["HT"] <= 2e-6, errs


ROOMS = [(64, 64, 3), (64, 64, 40), (128, 128, 2), (32, 32, 2), (64, 16, 5), (64, 32, 5), (32, 16, 3), (16, 16, 2)]


@pytest.mark.parametrize("K,V,units", ROOMS)
def test_same_bits_on_a_smaller_workspace(K, V, units):
    """Every workspace size from the least accepted to the full query: same outputs, bit for bit."""
    import torch
    T, N = 261, 1   # (V = 16 and 32 are split from some length on)
    print("case", K, V, units, flush=True)
    dev = gu.to_device(make_inputs(Workload("t", units, T, N, K, V, "bf16", 5, K ** -0.5, 1.0, use_H0=True)), "bf16")
    desc = mb.make_desc(units, T, N, K, V, mb.M2RNN_BF16)
    full = mb.m2rnn_workspace_bytes(desc, 0)
    part = units * T * N * V * 4
    w_r = torch.full((N, V), 0.5, dtype=torch.bfloat16, device="cuda")
    outs = []
    assert full >= 2 * part
    for P in [full // part] + [p for p in (8, 4, 2, 1) if p * part < full]:
        y = torch.full((units, T, N, V), float("nan"), dtype=torch.bfloat16, device="cuda")
        HT = torch.full((units, N, K, V), float("nan"), dtype=torch.float32, device="cuda")
        ws = torch.empty(max(P * part + 255, 256) // 256 * 256, dtype=torch.uint8, device="cuda")
        rc = mb.m2rnn_fwd_opt(desc, mb.make_opts(w_r=w_r), dev["q"], dev["k"], dev["v"], dev["f"], dev["W"],
                              dev["H0"], y, HT, None, ws, stream=torch.cuda.current_stream().cuda_stream, check=False)
        torch.cuda.synchronize()
        if rc != 0:
            assert rc == 5 and outs   # below the least: refused before a launch
            break
        outs.append((y, HT))
    for y, HT in outs[1:]:
        assert torch.equal(y, outs[0][0]) and torch.equal(HT, outs[0][1])
