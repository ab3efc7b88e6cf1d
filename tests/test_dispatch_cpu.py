"""CPU-only: which kernels a call launches and what memory they are handed, taken from the library
itself with a recorder in the place of the HIP runtime (tests/launch_recorder.py)."""
import pytest

from paper_2603_14360_amd import binding as mb
import launch_recorder as lr

WS = 0x10000000
BF16, F32 = mb.M2RNN_BF16, mb.M2RNN_F32


def d(B, T, N, K, V, io, **kw):
    return dict(B=B, T=T, N=N, K=K, V=V, io=io, **kw)


def ws_bytes(desc, bwd):
    return mb.m2rnn_workspace_bytes(mb.make_desc(**desc), bwd)


# every shape with a split forward that can also do without a workspace
NO_WORKSPACE = [(64, 32, 4), (64, 32, 70), (32, 16, 3), (32, 16, 200), (32, 32, 300), (16, 16, 40), (64, 64, 600)]


@pytest.mark.parametrize("K,V,units", NO_WORKSPACE)
def test_a_missing_workspace_is_never_written(K, V, units):
    """workspace = NULL with a size beside it (an allocation that failed, say): where the call can
    do without a workspace it takes a split without partial sums."""
    desc = d(units, 40, 1, K, V, BF16)
    null, none, full = lr.launches([dict(call="fwd", desc=desc, ws=None, ws_bytes=1 << 30),
                                    dict(call="fwd", desc=desc, ws=None, ws_bytes=0),
                                    dict(call="fwd", desc=desc, ws=WS, ws_bytes=1 << 30)])
    assert null["rc"] == none["rc"] == full["rc"] == 0
    assert null["launches"] == none["launches"]
    assert [l["kernel"].split("<")[0] for l in null["launches"]] in (["half_fwd_kernel"], ["rowwave_fwd_kernel"])
    for l in full["launches"]:
        assert l["partial"] in (None, WS)


def one_workgroup_per_state(desc, bwd):
    """Scratch of the fp32 scan with one workgroup per state: W and its transpose in fp32, and
    backward a chunk's states, a dW per state and, for shared heads, dq and dk of every head."""
    a = lambda x: (x + 255) // 256 * 256
    B, T, N, K, V = (desc[k] for k in "BTNKV")
    C = desc.get("chunk") or mb.m2rnn_default_chunk(mb.make_desc(**desc))
    n = 2 * a(N * V * V * 4)
    if bwd:
        heads = a(B * T * N * K * 4) if desc.get("Nqk", N) != N else 0
        n += a(B * N * (C + 1) * K * V * 4) + a(B * N * V * V * 4) + 2 * heads
        n += a(1024 * N * V * 4) + a(256 * 2 * N * 4)   # sums of the options' gradients
    return n


IN_TURN = [(K, V, io) for K, V in ((128, 16), (64, 32), (128, 32), (32, 64), (64, 64), (128, 64)) for io in (F32, BF16)]


@pytest.mark.parametrize("K,V,io", IN_TURN)
@pytest.mark.parametrize("B,T,N,chunk,Nqk", [(8, 4096, 16, 0, 16), (1, 65536, 32, 1, 32), (2, 100, 4, 256, 2), (3, 5000, 4, 17, 1)])
def test_fp32_kernels_without_room_for_partial_sums(K, V, io, B, T, N, chunk, Nqk):
    """The fp32 kernels of V <= 64 accept what one workgroup per state takes and then run the parts
    of a state in turn; below that they refuse."""
    desc = d(B, T, N, K, V, io, chunk=chunk, Nqk=Nqk)
    for call in ("fwd", "bwd"):
        bwd = int(call == "bwd")
        if mb.m2rnn_route_string(mb.make_desc(**desc), bwd)[:4] not in ("gene", "quad"):
            continue   # (bf16 io: matrix-core kernels)
        least, full = one_workgroup_per_state(desc, bwd), ws_bytes(desc, bwd)
        c = dict(call=call, desc=desc, ws=WS, ckpt=1, opts=1)
        under, at, query = lr.launches([dict(c, ws_bytes=min(least, full) - 1), dict(c, ws_bytes=least), dict(c, ws_bytes=full)])
        assert under["rc"] == 5 and not under["launches"]
        assert at["rc"] == 0 and query["rc"] == 0
        kern = [r["launches"][0] for r in (at, query)]
        assert kern[1]["kernel"].startswith("quad_%s_kernel" % call)
        if bwd:   # ... and without the forward's checkpoints, with room for them on top
            ck = (mb.m2rnn_ckpt_bytes(mb.make_desc(**desc)) + 255) // 256 * 256
            c = dict(c, ckpt=0)
            short, enough = lr.launches([dict(c, ws_bytes=min(least, full) + ck - 1), dict(c, ws_bytes=least + ck)])
            assert short["rc"] == 5 and enough["rc"] == 0 and enough["launches"][-1] == at["launches"][-1]
        if full > least:
            assert kern[0]["kernel"] == kern[1]["kernel"].replace(", false>", ", true>")
            assert kern[0]["grid"] == B * N and kern[1]["grid"] == B * N * (K * V // 1024)


SHAPES = [(64, 64, 84), (64, 64, 4), (128, 128, 8), (32, 32, 8), (16, 16, 3), (64, 16, 84), (64, 32, 8), (32, 16, 8),
          (128, 32, 4), (64, 128, 4)]


@pytest.mark.parametrize("io", [BF16, F32])
@pytest.mark.parametrize("K,V,N", SHAPES)
@pytest.mark.parametrize("B,T", [(4, 777), (1, 512)])
def test_backward_without_checkpoints_needs_room_for_them_and_no_more(K, V, N, B, T, io):
    """The pass that recomputes checkpoints writes no y: it adds the checkpoints to what the backward
    takes with the forward's, and nothing for partial sums of y."""
    desc = d(B, T, N, K, V, io)
    ck = (mb.m2rnn_ckpt_bytes(mb.make_desc(**desc)) + 255) // 256 * 256
    need = ws_bytes(desc, 2)
    assert need == ws_bytes(desc, 1) + ck
    (got,) = lr.launches([dict(call="bwd", desc=desc, ws=WS, ws_bytes=need)])
    assert got["rc"] == 0
    assert not any("y_parts_sum" in l["kernel"] for l in got["launches"])


# states around the lines of the forward's choice between the 8-row kernel and the 16-row ones
CHOICE = [(32, 32, 512, "half"), (32, 32, 513, "mfma"), (32, 32, 1023, "mfma"), (32, 32, 1024, "rowwave"), (64, 32, 384, "half"), (64, 32, 385, "rowwave"),
          (64, 32, 511, "rowwave"), (64, 32, 512, "rowwave"), (32, 16, 1023, "half"), (32, 16, 1024, "rowwave"),
          (64, 64, 511, "half"), (64, 64, 512, "rowwave"), (64, 16, 511, "half"), (64, 16, 512, "rowwave"),
          (16, 16, 2047, "half"), (16, 16, 2048, "rowwave"), (128, 128, 16, "half"), (128, 128, 17, "mfma")]


CHOICE = [c + (40,) for c in CHOICE] + [(64, 32, 256, "half", 2), (64, 32, 257, "rowwave", 31), (64, 32, 257, "half", 32)]


@pytest.mark.parametrize("K,V,units,kernel,T", CHOICE)
def test_forward_kernel_choice(K, V, units, kernel, T):
    """The kernel follows from the shape, the states and the steps alone; the workspace decides at most
    between splits of the same kernel (whose bits are the same), and the query is what the choice needs."""
    desc = d(units, T, 1, K, V, BF16)
    full = ws_bytes(desc, 0)
    calls = [dict(call="fwd", desc=desc, ws=WS, ws_bytes=n) for n in {full, 0, full + 4096, 1 << 40}]
    for r in lr.launches(calls):
        assert r["rc"] in (0, 5)
        if r["rc"] == 0:
            assert r["launches"][0]["kernel"].startswith(kernel + "_fwd_kernel")
    (r,) = lr.launches([dict(call="fwd", desc=desc, ws=WS, ws_bytes=full)])
    assert r["rc"] == 0


# states on both sides of the line between the 8-row forwards on waves that share a row's columns and on waves
# with whole rows; the choice looks at the shape and the states alone
WHOLE_ROWS = [(64, 64, 1, "Pair"), (64, 64, 32, "Pair"), (64, 64, 33, "Half"), (32, 32, 1, "Pair"), (32, 32, 128, "Pair"),
              (32, 32, 129, "Half"), (64, 32, 1, "Half"), (64, 32, 64, "Half"), (64, 16, 1, "Half"), (128, 128, 1, "Half")]


@pytest.mark.parametrize("K,V,units,form", WHOLE_ROWS)
def test_forward_on_waves_with_whole_rows(K, V, units, form):
    for T in (2, 16, 44, 48, 600):
        desc = d(units, T, 1, K, V, BF16)
        full = ws_bytes(desc, 0)
        calls = [dict(call="fwd", desc=desc, ws=WS, ws_bytes=n) for n in sorted({0, full // 4, full // 2, full})]
        got = lr.launches(calls + [dict(call="static", desc=desc), dict(call="bwd", desc=desc, ws=WS, ws_bytes=ws_bytes(desc, 2))])
        assert got[len(calls) - 1]["rc"] == got[-1]["rc"] == 0
        for r in got:
            assert r["rc"] in (0, 5)
            for k in (l["kernel"] for l in r["launches"]):
                assert not k.startswith("half_fwd_kernel") or "%s<%d, %d, " % (form, K, V) in k, (T, k)


HALF_SHAPES = [(64, 64), (128, 128), (32, 32), (16, 16), (64, 16), (32, 16), (64, 32)]


@pytest.mark.parametrize("K,V", HALF_SHAPES)
def test_every_split_that_is_chosen_is_built(K, V):
    """Any number of states around the lines, any room, any length: a launch or a refusal, and in the
    end the pass that recomputes checkpoints; never an instantiation that is missing."""
    lines = [1, 2, 4, 8, 16, 32, 64, 128, 256, 512, 1024, 2048]
    calls = []
    for units in sorted({max(1, u + e) for u in lines for e in (-1, 0, 1)}):
        for T in (2, 17, 46, 300):
            desc = d(units, T, 1, K, V, BF16)
            part = units * T * V * 4
            calls += [dict(call="fwd", desc=desc, ws=WS, ws_bytes=P * part) for P in (16, 8, 4, 2, 1, 0)]
            calls += [dict(call="static", desc=desc), dict(call="bwd", desc=desc, ws=WS, ws_bytes=ws_bytes(desc, 2))]
    for c, r in zip(calls, lr.launches(calls)):
        assert r["rc"] in (0, 5) and (r["rc"] == 0) == bool(r["launches"]), (c, r)


# fp32 kernels of V = 32: states and steps around the lines from which on, and up to which, rows are split
SPLIT_ROWS = [(32, 128, 16, "Split"), (32, 129, 16, "Quad"), (32, 8, 15, "Quad"), (32, 1, 1, "Quad"), (16, 256, 2, "Split"),
              (16, 257, 2, "Quad"), (16, 8, 1, "Quad"), (64, 8, 40, "Quad"), (128, 2, 40, "Quad")]


@pytest.mark.parametrize("K,units,T,form", SPLIT_ROWS)
def test_rows_are_split_where_that_pays(K, units, T, form):
    desc = d(units, T, 1, K, 32, F32)
    calls = [dict(call=c, desc=desc, ws=WS, ws_bytes=ws_bytes(desc, int(c == "bwd")), ckpt=1) for c in ("fwd", "bwd")]
    for r in lr.launches(calls):
        kernel = r["launches"][0]["kernel"]
        assert r["rc"] == 0 and "%s<%d, 32>" % (form, K) in kernel, kernel
    if K == 32 and form == "Quad":   # nothing is asked for what is not used
        assert ws_bytes(desc, 0) == 256


@pytest.mark.parametrize("T,N,split", [(8192, 32, True), (8193, 32, False), (65536, 32, False), (2048, 128, True), (65536, 4, True)])
def test_the_room_that_split_rows_ask_for_is_bounded(T, N, split):
    desc = d(1, T, N, 32, 32, F32)
    most, states = 64 << 20, N * 32 * 32 * 4
    fwd, bwd = ws_bytes(desc, 0), ws_bytes(desc, 1)
    assert fwd == (8 * N * T * 32 if split else 256) and fwd <= most
    # (backward: dv as y, df, a dW per workgroup and the sums of the options' gradients)
    assert bwd <= fwd + fwd // 32 + 2 * states + 4096 * N * 32 + 2048 * N + 1024
    for r in lr.launches([dict(call=c, desc=desc, ws=WS, ws_bytes=n, ckpt=1) for c, n in (("fwd", fwd), ("bwd", bwd))]):
        assert r["rc"] == 0 and ("Split<" in r["launches"][0]["kernel"]) == split


SCAN_KERNELS = ("half_fwd", "mfma_fwd", "rowwave_fwd", "quad_fwd", "gen_fwd", "decode", "mfma_bwd_overlap", "rowwave_bwd",
                "quad_bwd", "gen_bwd")


def test_every_scan_kernel_has_a_parity_case():
    """Every kernel of the scan that is compiled into the library is launched by a case of the GPU
    parity tests, and the route string of each case names the kernel that runs."""
    import test_gpu_half_fwd as half
    import test_gpu_instantiations as inst
    import test_gpu_quad_f32 as quad

    calls, routes = [], []

    def add(desc, bwd=False, room=None, route=None, **kw):
        n = ws_bytes(desc, (1 if kw.get("ckpt") else 2) if bwd else 0) if room is None else room
        calls.append(dict(call="bwd" if bwd else "fwd", desc=desc, ws=WS, ws_bytes=n, **kw))
        routes.append(mb.m2rnn_route_string(mb.make_desc(**desc), int(bwd)) if route is None else route)

    for K, V, B, N, Nqk, fr, br in inst.CASES:
        desc = d(B, 35, N, K, V, BF16, Nqk=Nqk or N)
        add(desc, route=fr, ckpt=1)
        add(desc, bwd=True, route=br, ckpt=1)
        add(desc, bwd=True, route="")
    for K, V, B, N, Nqk, fr, br in inst.CLIPPED:
        add(d(B, 35, N, K, V, BF16, Nqk=Nqk or N), bwd=True, route=br, ckpt=1, opts=1)
    for K, V, B, N, T, route in inst.SPLITS:
        add(d(B, T, N, K, V, BF16), route=route)
    for K, V, units in inst.CHECKPOINT_PASS:
        add(d(units, 35, 1, K, V, BF16), bwd=True, route="")
    for K, V in inst.DECODE:
        add(d(5, 1, 3, K, V, BF16))
    for K, V in inst.GENERIC_F32 + quad.SHAPES:
        add(d(2, 35, 3, K, V, F32), ckpt=1)
        add(d(2, 35, 3, K, V, F32), bwd=True, ckpt=1)
    for K, V in quad.SHAPES:
        add(d(2, 35, 3, K, V, F32), bwd=True, route="")
    for io, K, V, units in quad.MANY:
        desc = d(units, 35, 1, K, V, F32 if io == "f32" else BF16)
        add(desc, ckpt=1)
        add(desc, bwd=True, ckpt=1)
        add(desc, bwd=True, route="")
    for io, K, V, T, chunk, Nqk in quad.TURNS:
        desc = d(1, T, 4, K, V, F32 if io == "f32" else BF16, chunk=chunk, Nqk=Nqk)
        assert one_workgroup_per_state(desc, 1) < ws_bytes(desc, 1)
        add(desc, bwd=True, route="", ckpt=1, room=one_workgroup_per_state(desc, 1))
    for io, K, V in quad.FORWARD_TURNS:
        desc = d(1, 601, 16, K, V, F32)
        add(desc, route="", room=min(one_workgroup_per_state(desc, 0), ws_bytes(desc, 0)))
    for K, V, units in half.ROOMS:
        desc = d(units, 261, 1, K, V, BF16)
        for P in (16, 8, 4, 2, 1):
            add(desc, route="", room=P * units * 261 * V * 4)

    seen = set()
    for c, route, r in zip(calls, routes, lr.launches(calls)):
        assert r["rc"] in ((0, 5) if route == "" else (0,)), (c, r)
        names = [l["kernel"] for l in r["launches"]]
        scan = [n for n in names if n.split("_kernel")[0] in SCAN_KERNELS]
        seen |= set(scan)
        if route:
            family, shape = route[:-1].split("<")
            want = {"tile": "mfma_bwd_overlap" if c["call"] == "bwd" else "mfma_fwd", "half": "half_fwd", "rowwave": "rowwave_fwd",
                    "rowwave_bwd": "rowwave_bwd", "decode": "decode", "generic": "gen_" + c["call"], "quad": "quad_" + c["call"]}[family]
            assert len(scan) == 1 and scan[0].startswith(want + "_kernel<"), (route, scan)
            if family in ("tile", "half", "rowwave", "decode", "quad"):
                assert "<%s>" % shape.replace(",", ", ") in scan[0], (route, scan)
    every = {k for k in lr.kernels() if k.split("_kernel")[0] in SCAN_KERNELS}
    assert len(every) > 100 and not every - seen, sorted(every - seen)
