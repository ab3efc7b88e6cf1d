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


# many sequences of a few steps: more segments than workgroup rows, several to a walker
@pytest.mark.parametrize("io", ["f32", "bf16"])
@pytest.mark.parametrize("B,T,C", [(4200, 1, 1024), (2300, 3, 1016), (4096, 4, 520)])
def test_conv_many_short_sequences(io, B, T, C):
    conv_case(io, B, T, C, True)


# the longer segments, taken by launches that fill the chip: 16, 32 and 64 steps, ragged ends
@pytest.mark.parametrize("B,T,C,bias", [(3, 1399, 4000, True), (3, 2799, 4000, False), (17, 3901, 1024, True)])
def test_conv_long_segments(B, T, C, bias):
    conv_case("bf16", B, T, C, bias)


@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_a_nan_stays_where_it_belongs(io):
    """A NaN reaches the outputs that depend on it and no other: lanes and rows that a launch
    only pads with clamped loads must not leak into sums or neighbours."""
    import torch
    from paper_2603_14360_amd import binding as mb
    print("case nan", io, flush=True)
    B, T, C = 2, 70, 1048   # a last wave (norm) and a last workgroup (conv) that are nearly empty
    g = torch.Generator(device="cuda").manual_seed(3)
    dt = torch.float32 if io == "f32" else torch.bfloat16
    x, a, dout = (torch.randn(B, T, C, generator=g, device="cuda").to(dt) for _ in range(3))
    w4, b4, w = (torch.randn(*s, generator=g, device="cuda").to(dt) for s in ((C, 4), (C,), (C,)))
    st = torch.cuda.current_stream().cuda_stream

    def run(x):
        out, dx, o2, dy, da = (torch.empty_like(x) for _ in range(5))
        dw, db, dw2, s = (torch.empty(sh, device="cuda") for sh in ((C, 4), (C,), (C,), (B, T)))
        ws = torch.empty(max(mb.m2rnn_conv_silu_workspace_bytes(B, T, C), mb.m2rnn_gated_rmsnorm_workspace_bytes(B, T, C)),
                         dtype=torch.uint8, device="cuda")
        mb.m2rnn_conv_silu_fwd(x, w4, b4, out, stream=st)
        mb.m2rnn_conv_silu_bwd(x, w4, b4, dout, dx, dw, db, ws, stream=st)
        mb.m2rnn_gated_rmsnorm_fwd(x, a, w, 1e-5, o2, s, stream=st)
        mb.m2rnn_gated_rmsnorm_bwd(x, a, w, 1e-5, s, dout, dy, da, dw2, ws, stream=st)
        return out, dx, dw, db, o2, dy, da, s

    clean = run(x)
    bad = x.clone()
    bad[0, 20, C - 1] = float("nan")
    # conv: the channel's next three steps and, backward, three steps around them; norm: the token
    hit = [torch.zeros_like(t, dtype=torch.bool) for t in clean]
    hit[0][0, 20:24, C - 1] = True
    hit[1][0, 17:24, C - 1] = True
    hit[2][C - 1] = True
    hit[3][C - 1] = True
    for i in (4, 5, 6, 7):
        hit[i][0, 20] = True
    for got, ref, h in zip(run(bad), clean, hit):
        assert torch.equal(got[~h], ref[~h])
        assert got[h].isnan().all()
