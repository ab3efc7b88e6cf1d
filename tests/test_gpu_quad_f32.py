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


# shapes whose rows are split between the halves of a wave as long as every wave has a SIMD for itself:
# the last launch that is split, the first that is not
MANY = [("f32", 32, 32, 128), ("f32", 32, 32, 129), ("f32", 16, 32, 256), ("f32", 16, 32, 258), ("bf16", 16, 32, 256),
        ("bf16", 16, 32, 258)]


@pytest.mark.parametrize("io,K,V,units", MANY)
def test_split_rows_and_whole_rows(io, K, V, units):
    """Both sides of the line, and the backward that recomputes the checkpoints: same bits as with them."""
    T = 35
    print("case split rows", io, K, V, units, flush=True)
    inp = make_inputs(Workload("t", units, T, 1, K, V, io, 90 + K + units, K ** -0.5, 1.0, use_H0=True, use_dHT=True))
    got, again = gu.run_gpu(inp, io), gu.run_gpu(inp, io, use_ckpt=False)
    gu.compare(got, gu.run_oracle(inp), gu.TOL[io], label="split rows")
    assert all((again[n] == got[n]).all() for n in got)


@pytest.mark.parametrize("fwd", [True, False])
def test_split_rows_need_no_more_room_than_whole_rows(fwd):
    """32 x 32, few states: finer parts are taken with room for their sums only; the room of one workgroup
    per state stays enough, and nothing is written behind it."""
    import torch
    from paper_2603_14360_amd import binding as mb
    B, T, N, K, V = 2, 53, 3, 32, 32
    desc = mb.make_desc(B, T, N, K, V, mb.M2RNN_F32)
    full = mb.m2rnn_workspace_bytes(desc, 0 if fwd else 1)
    al = lambda x: (x + 255) // 256 * 256
    # one workgroup per state: nothing forward; a dW per state backward, and the options' sums
    least = 256 if fwd else al(B * N * V * V * 4) + al(1024 * N * V * 4) + al(256 * 2 * N * 4)
    assert least < full
    print("case split rows, least room", fwd, flush=True)
    inp = make_inputs(Workload("t", B, T, N, K, V, "f32", 31, K ** -0.5, 1.0, use_H0=True, use_dHT=True))
    dev, ref = gu.to_device(inp, "f32"), gu.run_oracle(inp)
    scan = mb.Scan(B, T, N, K, V, "f32")
    args = [dev[n] for n in ("q", "k", "v", "f", "W", "H0")]
    scan.fwd(*args)
    new = lambda *s: torch.full(s, float("nan"), device="cuda")
    for n in (full, least):
        ws = torch.full((n + 4096,), 0xFF, dtype=torch.uint8, device="cuda")   # (a guard behind the workspace)
        stream = torch.cuda.current_stream().cuda_stream
        if fwd:
            names, out = ("y", "HT"), [new(B, T, N, V), new(B, N, K, V)]
            mb.m2rnn_fwd_opt(desc, mb.make_opts(), *args, *out, None, ws[:n], stream=stream)
        else:
            names = gu.GRAD_NAMES
            out = [new(B, T, N, K), new(B, T, N, K), new(B, T, N, V), new(B, T, N), new(N, V, V), new(B, N, K, V)]
            mb.m2rnn_bwd_opt(desc, mb.make_opts(), *args, scan.ckpt, dev["dy"], dev["dHT"], *out, ws[:n], stream=stream)
        torch.cuda.synchronize()
        assert (ws[n:] == 0xFF).all()
        got = {name: gu.to_np(x) for name, x in zip(names, out)}
        gu.compare(got, {name: ref[name] for name in got}, gu.TOL["f32"], label="room %d" % n)


def test_split_rows_give_the_bits_of_whole_rows():
    """32 x 32: neither the room nor the entry point shows in y, H_T or the checkpoints, nor, in the
    backward, in what comes from the carried gradient; a pass that recomputes its checkpoints follows the
    forward's trajectory on any room."""
    import torch
    from paper_2603_14360_amd import binding as mb
    B, T, N, K, V = 2, 53, 3, 32, 32
    desc = mb.make_desc(B, T, N, K, V, mb.M2RNN_F32)
    al = lambda x: (x + 255) // 256 * 256
    print("case split rows, bits", flush=True)
    inp = make_inputs(Workload("t", B, T, N, K, V, "f32", 32, K ** -0.5, 1.0, use_H0=True, use_dHT=True))
    dev = gu.to_device(inp, "f32")
    args = [dev[n] for n in ("q", "k", "v", "f", "W", "H0")]
    w_r, stream = torch.randn(N, V, device="cuda"), torch.cuda.current_stream().cuda_stream
    new = lambda *s: torch.full(s, float("nan"), device="cuda")
    room = lambda n: torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
    outs = []
    for n in (mb.m2rnn_workspace_bytes(desc, 0), 256, None):
        out = [new(B, T, N, V), new(B, N, K, V), new(mb.m2rnn_ckpt_bytes(desc) // 4)]
        opts = mb.make_opts(w_r=w_r)
        if n is None:
            mb.m2rnn_fwd_static(desc, opts, *args, *out, stream=stream)
        else:
            mb.m2rnn_fwd_opt(desc, opts, *args, *out, room(n), stream=stream)
        outs.append(out)
    ckpt = outs[0][2]
    least = al(B * N * V * V * 4) + al(1024 * N * V * 4) + al(256 * 2 * N * 4)
    grads = []
    for n, own in ((mb.m2rnn_workspace_bytes(desc, 1), 0), (least, 0), (least, al(ckpt.numel() * 4))):
        out = [new(B, T, N, K), new(B, T, N, K), new(B, T, N, V), new(B, T, N), new(N, V, V), new(B, N, K, V)]
        mb.m2rnn_bwd_opt(desc, mb.make_opts(), *args, None if own else ckpt, dev["dy"], dev["dHT"], *out, room(n + own),
                         stream=stream)
        grads.append(out)
    torch.cuda.synchronize()
    for out in outs:
        assert all(torch.equal(a, b) and torch.isfinite(a).all() for a, b in zip(out, outs[0]))
    assert all(torch.equal(a, b) and torch.isfinite(a).all() for a, b in zip(grads[1], grads[2]))
    for name, a, b in zip(gu.GRAD_NAMES, grads[0], grads[1]):
        assert name not in ("dq", "dk", "dH0") or torch.equal(a, b), name


@pytest.mark.parametrize("K,most", [(32, 128), (16, 256)])
def test_bits_do_not_depend_on_the_number_of_states(K, most):
    """The last launch that is split and the first that is not: the same states, the same bits."""
    import torch
    from paper_2603_14360_amd import binding as mb
    T, V = 35, 32
    print("case split rows, states", K, most, flush=True)
    dev = gu.to_device(make_inputs(Workload("t", most + 1, T, 1, K, V, "f32", 33, K ** -0.5, 1.0, use_H0=True, use_dHT=True)), "f32")
    outs = []
    for B in (most + 1, most):
        args = [dev[n] if n == "W" else dev[n][:B].contiguous() for n in ("q", "k", "v", "f", "W", "H0")]
        scan = mb.Scan(B, T, 1, K, V, "f32")
        y, HT = scan.fwd(*args)
        g = scan.bwd(*args, dev["dy"][:B].contiguous(), dev["dHT"][:B].contiguous())
        outs.append([x[:most].clone() for x in (y, HT, g[0], g[1], g[5])])
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*outs))


FORWARD_TURNS = [("f32", K, V) for K, V in ((128, 16), (64, 32), (128, 32), (32, 64), (64, 64), (128, 64))]


@pytest.mark.parametrize("io,K,V", FORWARD_TURNS)
def test_parts_in_turn_give_the_same_bits(io, K, V):
    """The parts of a state one after the other against the side-by-side kernel on a full workspace:
    on the room of one workgroup per state, and m2rnn_fwd_static with partial sums larger than its scratch."""
    import torch
    from paper_2603_14360_amd import binding as mb
    B, T, N = 1, 601, 16
    desc = mb.make_desc(B, T, N, K, V, mb.M2RNN_F32)
    need = mb.m2rnn_workspace_bytes(desc, 0)
    print("case fp32 forward in turn", K, V, flush=True)
    inp = make_inputs(Workload("t", B, T, N, K, V, "f32", 9, K ** -0.5, 1.0, use_H0=True))
    dev = gu.to_device(inp, "f32")
    stream = torch.cuda.current_stream().cuda_stream
    w_r = torch.randn(N, V, device="cuda")
    rooms = [need, (2 * N * V * V * 4 + 511) // 512 * 512]
    if (K, V) == (64, 64):
        assert need > mb.M2RNN_STATIC_SCRATCH_BYTES
        rooms.append(None)
    outs = []
    for room in rooms:
        y, HT = torch.full((B, T, N, V), float("nan"), device="cuda"), torch.empty(B, N, K, V, device="cuda")
        ckpt = torch.full((mb.m2rnn_ckpt_bytes(desc) // 4,), float("nan"), device="cuda")
        args = (dev["q"], dev["k"], dev["v"], dev["f"], dev["W"], dev["H0"], y, HT, ckpt)
        if room is None:
            mb.m2rnn_fwd_static(desc, mb.make_opts(w_r=w_r), *args, stream=stream)
        else:
            ws = torch.empty(room, dtype=torch.uint8, device="cuda")
            mb.m2rnn_fwd_opt(desc, mb.make_opts(w_r=w_r), *args, ws, stream=stream)
        torch.cuda.synchronize()
        outs.append((y, HT, ckpt))
    for out in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(outs[0], out))
    assert all(torch.isfinite(a).all() for a in outs[0])


# long enough that the query is more than the room of one workgroup per state; checkpoint intervals
# below, at and above the 16 steps that stay on chip, ragged ends
TURNS = [(128, 16, 1300, 17, 2), (128, 16, 300, 1, 4), (64, 32, 300, 3, 4), (64, 32, 700, 17, 2), (128, 32, 650, 16, 1),
         (32, 64, 330, 0, 2), (64, 64, 330, 17, 4), (64, 64, 700, 33, 4), (128, 64, 330, 5, 2)]
# (bf16 io: the shapes without a matrix-core backward)
TURNS = [("f32",) + c for c in TURNS] + [("bf16",) + c for c in TURNS if c[:2] not in ((128, 16), (64, 64))]


@pytest.mark.parametrize("io,K,V,T,chunk,Nqk", TURNS)
def test_backward_parts_in_turn(io, K, V, T, chunk, Nqk):
    """A workspace without room for the partial sums of a state's parts: the parts one after the other
    against the side-by-side kernel and the oracle.  Only dW is added in another order."""
    import torch
    from paper_2603_14360_amd import binding as mb
    B, N = 1, 4
    desc = mb.make_desc(B, T, N, K, V, mb.M2RNN_F32 if io == "f32" else mb.M2RNN_BF16, Nqk=Nqk, chunk=chunk)
    print("case in turn", io, K, V, T, chunk, Nqk, flush=True)
    C = chunk or mb.m2rnn_default_chunk(desc)
    full = mb.m2rnn_workspace_bytes(desc, 1)
    al = lambda x: (x + 255) // 256 * 256
    inp = make_inputs(Workload("t", B, T, N, K, V, io, 9 + K + T, K ** -0.5, 1.0, use_H0=True, use_dHT=True, Nqk=Nqk))
    dev = gu.to_device(inp, io)
    dt = torch.float32 if io == "f32" else torch.bfloat16
    w_r = torch.linspace(-1, 1, N * V, device="cuda").reshape(N, V).to(dt)
    scan = mb.Scan(B, T, N, K, V, io, Nqk=Nqk, chunk=chunk)
    args = [dev[n] for n in ("q", "k", "v", "f", "W", "H0")]
    scan.fwd(*args, w_r=w_r)
    # the least: the layout of one workgroup per state, and what sits behind it
    least = 2 * al(N * V * V * 4) + al(B * N * (C + 1) * K * V * 4) + al(B * N * V * V * 4)
    least += (2 * al(B * T * N * K * 4) if Nqk != N else 0) + al(1024 * N * V * 4) + al(256 * 2 * N * 4)
    assert least < full
    outs = []
    for n in (full, least):
        new = lambda *s, dtype=torch.float32: torch.full(s, float("nan"), dtype=dtype, device="cuda")
        g = [new(B, T, Nqk, K, dtype=dt), new(B, T, Nqk, K, dtype=dt), new(B, T, N, V, dtype=dt), new(B, T, N),
             new(N, V, V), new(B, N, K, V)]
        dw_r = new(N, V)
        ws = torch.full((n + 4096,), 0xFF, dtype=torch.uint8, device="cuda")   # (a guard behind the workspace)
        mb.m2rnn_bwd_opt(desc, mb.make_opts(w_r, dw_r, 0.7), *args, scan.ckpt, dev["dy"], dev["dHT"], *g, ws[:n],
                         stream=torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        assert (ws[n:] == 0xFF).all()
        outs.append(g + [dw_r])
    ref = gu.run_oracle(dict(inp, w_r=w_r.double().cpu().numpy()), grad_clip=0.7)
    for g in outs:
        got = {name: gu.to_np(x) for name, x in zip(gu.GRAD_NAMES + ("dw_r",), g)}
        gu.compare(got, {n: ref[n] for n in got}, gu.TOL[io], label="in turn")
    for name, x, y in zip(gu.GRAD_NAMES, outs[0], outs[1]):
        assert name == "dW" or torch.equal(x, y), name
