"""The calls that a user of the library has it do, as cases to be timed.

Five kinds, all through `paper_2603_14360_amd.binding` as a program with torch tensors calls it:

  decode    one token per call: the recurrent form of inference, the state handed in and out
  prefill   forward over a prompt, no checkpoints
  train     forward (writing checkpoints) and backward of the scan
  conv      causal conv1d(4) + SiLU in front of the scan, forward and backward
  norm      gated RMSNorm behind the scan, forward and backward

Sizes are those of the benchmark's workloads and of the paper's layer (K = 64, V = 16, 84 heads
with one shared q/k head), together with odd lengths, other state sizes and the options of the
layer.  W is drawn as a layer that trains stably has it: part of the identity that it is initialised
to and a random part, with a largest singular value near one.  (With a larger one some of the many
recurrences are chaotic over thousands of steps, and two correct evaluations differ without bound.)
Gates are those of a layer with a memory of some ten steps: logits N(2, 1).
"""
import math

import torch

from paper_2603_14360_amd import binding as mb

_DT = {"bf16": torch.bfloat16, "f32": torch.float32}
_EPS = 1e-5


def _scan(kind, B, T, N, K, V, Nqk=0, io="bf16", gate=False, residual=False, carry=False, clip=0.0,
          name=None):
    """gate: psi(x) inside the library; residual: w_r (.) v_t; carry: an initial state is given
    (and, in training, the gradient of the final one); clip: per-step gradient clipping."""
    c = {"kind": kind, "B": B, "T": T, "N": N, "Nqk": Nqk or N, "K": K, "V": V, "io": io,
         "gate": gate, "residual": residual, "carry": carry, "clip": clip}
    return c if name is None else dict(c, name=name)


def _block(kind, B, T, C, io="bf16", bias=False, name=None):
    c = {"kind": kind, "B": B, "T": T, "C": C, "io": io, "bias": bias}
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # one sequence served token by token through the paper's layer: a single launch
        _scan("decode", 1, 1, 84, 64, 16, Nqk=1, gate=True, residual=True, carry=True,
              name="decode_one"),
        # a large serving batch, 64 x 64 states: the state's traffic
        _scan("decode", 256, 1, 16, 64, 64, carry=True, name="decode_batch"),
        # a few prompts of odd length through the paper's layer
        _scan("prefill", 4, 777, 84, 64, 16, Nqk=1, gate=True, residual=True, name="prefill_prompts"),
        # one long document on few states (benchmark workload C5)
        _scan("prefill", 1, 65536, 32, 64, 64, name="prefill_long"),
        # training steps of the benchmark: the headline (C3), the large state (C4), the paper's
        # layer (P1)
        _scan("train", 8, 4096, 16, 64, 64, name="train_headline"),
        _scan("train", 4, 8192, 8, 128, 128, name="train_wide"),
        _scan("train", 8, 4096, 84, 64, 16, Nqk=1, name="train_layer"),
        # many short sequences of odd length with everything that the layer can switch on
        _scan("train", 32, 1000, 16, 64, 64, gate=True, residual=True, carry=True, clip=1.0,
              name="train_segments"),
        # a small model in a unit test or an ablation: launches and latency
        _scan("train", 2, 333, 8, 32, 32, carry=True, name="train_small"),
        # fp32 storage, for debugging and for comparing with another implementation (C2)
        _scan("train", 4, 512, 8, 32, 32, io="f32", carry=True, name="train_fp32"),
        # the scan's neighbours at the widths of the paper's layer: q, k and v channels, and N V
        _block("conv", 8, 4096, 64 + 64 + 84 * 16, bias=True, name="conv_train"),
        _block("norm", 8, 4096, 84 * 16, name="norm_train"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# State elements times steps that one drawn scan may have: those of the headline's training step.
# Training in fp32, and of states whose sides differ, is the work of small experiments: at most
# 256 states, and T K V^2 of seven times the listed fp32 case.
_MAX_ELEMENT_STEPS = 8 * 16 * 4096 * 64 * 64
_MAX_SMALL = 7 * 512 * 32 ** 3


def draw(rng):
    kind = rng.choice(["decode", "prefill", "prefill", "train", "train", "train", "train", "block", "block"])
    if kind == "block":
        return _block(rng.choice(["conv", "norm"]), rng.randint(1, 8), _log_int(rng, 100, 4096),
                      8 * _log_int(rng, 16, 256), io=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                      bias=rng.random() < 0.5)
    K, V = rng.choice([(64, 16), (64, 16), (64, 64), (64, 64), (32, 32), (128, 128), (16, 16), (128, 64), (64, 32)])
    layer = (K, V) == (64, 16)
    N = rng.choice([12, 21, 42, 84]) if layer else rng.choice([2, 4, 8, 12, 16, 32])
    opts = {"Nqk": 1 if layer else N, "gate": rng.random() < 0.5, "residual": rng.random() < 0.5,
            "carry": rng.random() < 0.5}
    if kind == "decode":
        return _scan("decode", _log_int(rng, 1, 256), 1, N, K, V, **dict(opts, carry=True))
    io = "f32" if kind == "train" and K <= 64 and rng.random() < 0.25 else "bf16"
    T, states = 16384 if kind == "prefill" else 4096, 32 * N
    if io == "f32" or (kind == "train" and (K, V) in ((128, 64), (64, 32))):
        T, states = min(512, _MAX_SMALL // (K * V * V)), 256
    T = _log_int(rng, 50, T)
    most = min(states, _MAX_ELEMENT_STEPS // (T * K * V)) // N
    return _scan(kind, _log_int(rng, 1, max(1, most)), T, N, K, V, io=io,
                 clip=rng.choice([0.0, 0.0, 1.0]) if kind == "train" else 0.0, **opts)


def _randn(g, *shape, scale=1.0, mean=0.0, dtype=torch.float32):
    x = torch.randn(shape, generator=g, device="cuda", dtype=torch.float32)
    return x.mul_(scale).add_(mean).to(dtype)


def _prepare_block(c, g):
    B, T, C, dt = c["B"], c["T"], c["C"], _DT[c["io"]]
    s = {"kind": c["kind"], "x": _randn(g, B, T, C, dtype=dt), "dout": _randn(g, B, T, C, dtype=dt)}
    new = lambda *shape: torch.empty(shape, device="cuda", dtype=torch.float32)
    s["out"], s["dx"] = torch.empty_like(s["x"]), torch.empty_like(s["x"])
    if c["kind"] == "conv":
        s["w"] = _randn(g, C, 4, scale=0.5, dtype=dt)
        s["bias"] = _randn(g, C, scale=0.5, dtype=dt) if c["bias"] else None
        s["dw"], s["dbias"] = new(C, 4), new(C) if c["bias"] else None
        nbytes = mb.m2rnn_conv_silu_workspace_bytes(B, T, C)
    else:
        s["a"] = _randn(g, B, T, C, dtype=dt)
        s["w"] = _randn(g, C, scale=0.1, mean=1.0, dtype=dt)
        s["da"], s["dw"], s["scale"] = torch.empty_like(s["x"]), new(C), new(B, T)
        nbytes = mb.m2rnn_gated_rmsnorm_workspace_bytes(B, T, C)
    s["workspace"] = torch.empty(max(nbytes, 256), dtype=torch.uint8, device="cuda")
    return s


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    c = case
    if c["kind"] in ("conv", "norm"):
        return _prepare_block(c, g)
    B, T, N, Nqk, K, V, dt = c["B"], c["T"], c["N"], c["Nqk"], c["K"], c["V"], _DT[c["io"]]
    train = c["kind"] == "train"
    s = {"kind": c["kind"], "clip": c["clip"]}
    s["q"] = _randn(g, B, T, Nqk, K, scale=K ** -0.5, dtype=dt)
    s["k"] = _randn(g, B, T, Nqk, K, scale=K ** -0.5, dtype=dt)
    s["v"] = _randn(g, B, T, N, V, scale=K ** -0.5, dtype=dt)
    logits = _randn(g, B, T, N, mean=2.0)
    if c["gate"]:
        # psi(x) = (1 + e^(x + beta))^(-alpha): near 0.85 for these inputs, as the gates below
        s["f"] = logits.sub_(2.0)
        s["gate"] = (_randn(g, N, scale=0.1, mean=0.9), _randn(g, N, scale=0.1, mean=-2.0))
    else:
        s["f"], s["gate"] = torch.sigmoid_(logits), None
    W = _randn(g, N, V, V, scale=0.25 * V ** -0.5)
    s["W"] = W.add_(torch.eye(V, device="cuda"), alpha=0.5).to(dt)
    s["H0"] = _randn(g, B, N, K, V, scale=0.1) if c["carry"] else None
    s["w_r"] = _randn(g, N, V, scale=0.5, mean=0.5, dtype=dt) if c["residual"] else None
    s["dy"] = _randn(g, B, T, N, V, dtype=dt) if train else None
    s["dHT"] = _randn(g, B, N, K, V, scale=0.1) if train and c["carry"] else None
    s["scan"] = mb.Scan(B, T, N, K, V, c["io"], Nqk=Nqk, backward=train)
    return s


def run(state):
    s = state
    if s["kind"] == "conv":
        stream = torch.cuda.current_stream().cuda_stream
        mb.m2rnn_conv_silu_fwd(s["x"], s["w"], s["bias"], s["out"], stream=stream)
        mb.m2rnn_conv_silu_bwd(s["x"], s["w"], s["bias"], s["dout"], s["dx"], s["dw"], s["dbias"],
                               s["workspace"], stream=stream)
        out = {"out": s["out"], "dx": s["dx"], "dw": s["dw"]}
        return out if s["dbias"] is None else dict(out, dbias=s["dbias"])
    if s["kind"] == "norm":
        stream = torch.cuda.current_stream().cuda_stream
        mb.m2rnn_gated_rmsnorm_fwd(s["x"], s["a"], s["w"], _EPS, s["out"], s["scale"], stream=stream)
        mb.m2rnn_gated_rmsnorm_bwd(s["x"], s["a"], s["w"], _EPS, s["scale"], s["dout"], s["dx"],
                                   s["da"], s["dw"], s["workspace"], stream=stream)
        return {"out": s["out"], "scale": s["scale"], "dy": s["dx"], "da": s["da"], "dw": s["dw"]}
    scan = s["scan"]
    y, HT = scan.fwd(s["q"], s["k"], s["v"], s["f"], s["W"], s["H0"], w_r=s["w_r"], gate=s["gate"])
    if s["kind"] != "train":
        return {"y": y, "HT": HT}
    grads = scan.bwd(s["q"], s["k"], s["v"], s["f"], s["W"], s["H0"], s["dy"], s["dHT"],
                     w_r=s["w_r"], grad_clip=s["clip"], gate=s["gate"])
    names = ["dq", "dk", "dv", "df", "dW", "dH0"]
    names += ["dw_r"] if s["w_r"] is not None else []
    names += ["dalpha", "dbeta"] if s["gate"] is not None else []
    return dict(zip(names, grads), y=y, HT=HT)


def work(case):
    """Bytes: every input once, every output once.  Flops: a multiplication or an addition each,
    a transcendental as one; no recomputation of the forward in the backward beyond Z itself."""
    c, io = case, 2 if case["io"] == "bf16" else 4
    if c["kind"] in ("conv", "norm"):
        n = c["B"] * c["T"] * c["C"]
        # conv: x, dout, out, dx; norm: y, a, dout, out, dy, da
        tensors, flops = (4, 45) if c["kind"] == "conv" else (6, 40)
        return {"bytes": n * io * tensors, "flops": n * flops}
    steps, state = c["B"] * c["T"], c["B"] * c["N"] * c["K"] * c["V"] * 4
    qk, v, f = steps * c["Nqk"] * c["K"] * io, steps * c["N"] * c["V"] * io, steps * c["N"] * 4
    W = c["N"] * c["V"] * c["V"]
    nbytes = 2 * qk + 2 * v + f + W * io + state * (2 if c["carry"] else 1)
    flops = 2 * c["V"] + 11
    if c["kind"] == "train":
        # dy in; dq, dk, dv, df, dW, dH0 out
        nbytes += 2 * qk + 2 * v + f + W * 4 + state * (2 if c["carry"] else 1)
        flops += 6 * c["V"] + 25
    return {"bytes": nbytes, "flops": flops * steps * c["N"] * c["K"] * c["V"]}


def tolerance(case):
    # Four times what the library shows against a 64-bit evaluation: bf16 outputs 1.7e-3 (their
    # rounding), fp32 outputs up to 6e-7 (sums over batch and steps, the longest of some 10^4 terms).
    return {"rel": 2.5e-6 if case["io"] == "f32" else 7e-3}
