"""CPU-only: the module that hands a Scan's tensors to the library.  What arrives there is read with a
recorder in the place of the library's entry points."""
import ctypes

import pytest
import torch

from paper_2603_14360_amd import binding as mb

P = ctypes.c_void_p
FWD = ctypes.CFUNCTYPE(ctypes.c_int, P, ctypes.POINTER(mb.m2rnn_opts), *[P] * 10, ctypes.c_size_t, P)
BWD = ctypes.CFUNCTYPE(ctypes.c_int, P, ctypes.POINTER(mb.m2rnn_opts), *[P] * 16, ctypes.c_size_t, P)


@pytest.fixture
def recorded():
    """(scan, calls): calls collects (name, options, arguments) instead of running them."""
    calls = []

    def record(name):
        def f(desc, opts, *args):
            calls.append((name, {n: getattr(opts[0], n) for n, _ in mb.m2rnn_opts._fields_}, (desc,) + args))
            return 0 if len(calls) < 9 else 3
        return f
    fwd, bwd = FWD(record("fwd")), BWD(record("bwd"))
    native, L = mb._call(), mb.lib()
    address = lambda f: ctypes.cast(f, P).value
    native.init(address(fwd), address(bwd))
    try:
        scan = mb.Scan(2, 3, 4, 16, 16, "bf16", device="cpu")
        scan._stream = lambda: 77
        yield scan, calls
    finally:
        native.init(address(L.m2rnn_fwd_opt), address(L.m2rnn_bwd_opt))


def test_arguments_reach_their_places(recorded):
    scan, calls = recorded
    t = lambda: torch.zeros(8)
    q, k, v, f, W, H0, dy, dHT, w_r, alpha, beta = (t() for _ in range(11))
    a = lambda x: x.data_ptr()
    ws, n = a(scan.workspace), scan.workspace.numel()
    none = dict.fromkeys(("w_r", "dw_r", "gate_alpha", "gate_beta", "dgate_alpha", "dgate_beta"), None)
    desc = ctypes.addressof(scan.desc)

    assert scan.fwd(q, k, v, f, W, H0) == (scan.y, scan.HT)
    args = tuple(map(a, (q, k, v, f, W, H0, scan.y, scan.HT, scan.ckpt))) + (ws, n, 77)
    assert calls[-1] == ("fwd", dict(none, grad_clip=0.0), (desc,) + args)
    scan.fwd(a(q), k, v, f, W, w_r=w_r, gate=(alpha, beta))   # (an address for a tensor; no H0)
    opts = dict(none, grad_clip=0.0, w_r=a(w_r), gate_alpha=a(alpha), gate_beta=a(beta))
    assert calls[-1] == ("fwd", opts, (desc,) + args[:5] + (None,) + args[6:])

    outs = (scan.dq, scan.dk, scan.dv, scan.df, scan.dW, scan.dH0)
    got = scan.bwd(q, k, v, f, W, H0, dy, dHT)
    assert all(x is y for x, y in zip(got, outs)) and len(got) == 6
    args = tuple(map(a, (q, k, v, f, W, H0, scan.ckpt, dy, dHT) + outs)) + (ws, n, 77)
    assert calls[-1] == ("bwd", dict(none, grad_clip=0.0), (desc,) + args)
    scan.bwd(q, k, v, f, W, H0, dy, grad_clip=-1.0)   # (off)
    assert calls[-1][1]["grad_clip"] <= 0.0 and calls[-1][2][9] is None
    got = scan.bwd(q, k, v, f, W, None, dy, dHT, use_ckpt=False, w_r=w_r, grad_clip=0.5, gate=(alpha, beta))
    assert [tuple(x.shape) for x in got[6:]] == [(4, 16), (4,), (4,)]
    opts = dict(w_r=a(w_r), dw_r=a(got[6]), grad_clip=0.5, gate_alpha=a(alpha), gate_beta=a(beta), dgate_alpha=a(got[7]),
                dgate_beta=a(got[8]))
    assert calls[-1] == ("bwd", opts, (desc,) + args[:5] + (None, None) + args[7:])


def test_whatever_has_an_address_is_taken(recorded):
    """As by the ctypes calls: a subclass of the tensor with a data_ptr of its own, a parameter, and any other
    object that has the method; its exceptions come through."""
    class Own(torch.Tensor):
        def data_ptr(self):
            return 4096

    class Buffer:
        def data_ptr(self):
            return 8192

    class Lost:
        def data_ptr(self):
            raise KeyError("lost")

    scan, calls = recorded
    x, w = torch.zeros(8), torch.nn.Parameter(torch.zeros(8))
    scan.fwd(torch.zeros(8).as_subclass(Own), Buffer(), x, x, w)
    assert calls[-1][2][1:6] == (4096, 8192, x.data_ptr(), x.data_ptr(), w.data_ptr())
    with pytest.raises(KeyError):
        scan.fwd(Lost(), x, x, x, w)


def test_errors_are_exceptions(recorded):
    scan, calls = recorded
    x = torch.zeros(8)
    with pytest.raises(TypeError):
        scan.fwd([0], x, x, x, x)
    with pytest.raises(RuntimeError):
        scan.fwd(torch.empty(2, layout=torch.sparse_coo), x, x, x, x)
    assert not calls
    with pytest.raises(TypeError):
        scan._native.fwd(x)
    calls.extend([None] * 9)
    with pytest.raises(mb.M2RNNError) as e:
        scan.fwd(x, x, x, x, x)
    assert e.value.code == 3 and "m2rnn_fwd failed" in str(e.value)
    with pytest.raises(mb.M2RNNError, match="m2rnn_bwd_opt failed"):
        scan.bwd(x, x, x, x, x, None, x, grad_clip=1.0)


@pytest.mark.parametrize("fault", ["no compiler", "no torch"])
def test_the_library_is_built_without_the_call_module(tmp_path, monkeypatch, fault):
    """A missing host compiler or torch leaves libm2rnn.so built and in its place."""
    import builtins
    from paper_2603_14360_amd import build
    (tmp_path / "a.hip").write_text("")
    for name, value in (("CSRC", tmp_path), ("OBJ", tmp_path / "o"), ("LIB", tmp_path / "lib.so"), ("CALL", tmp_path / "call.so")):
        monkeypatch.setattr(build, name, str(value))
    monkeypatch.setattr(build, "_compile", lambda src: src + ".o")
    monkeypatch.setattr(build.subprocess, "check_call", lambda cmd: open(cmd[cmd.index("-o") + 1], "w").close())
    if fault == "no compiler":
        monkeypatch.setattr(build, "CXX", str(tmp_path / "missing"))
        with pytest.raises(RuntimeError, match="py_call"):
            build.build(verbose=False)
    else:
        real = builtins.__import__

        def without_torch(name, *args, **kw):
            if name == "torch":
                raise ImportError(name)
            return real(name, *args, **kw)
        monkeypatch.setattr(builtins, "__import__", without_torch)
        assert build.build(verbose=False) == str(tmp_path / "lib.so")
    assert (tmp_path / "lib.so").exists() and not (tmp_path / "call.so").exists()


def test_a_call_module_of_another_torch_or_python_is_refused(monkeypatch):
    import sys
    import paper_2603_14360_amd as package
    module = mb._call()
    assert module.torch_version == torch.__version__ and module.__file__.endswith(".so") and "cpython" in module.__file__
    monkeypatch.setattr(mb, "_call_module", None)
    monkeypatch.setattr(torch, "__version__", "0.0")
    with pytest.raises(RuntimeError, match="this is 0.0; run"):
        mb._call()
    monkeypatch.undo()
    monkeypatch.setattr(mb, "_call_module", None)
    monkeypatch.delattr(package, "_call", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2603_14360_amd._call", None)   # (as where no file has this Python's name)
    with pytest.raises(RuntimeError, match="not built for this Python"):
        mb._call()


def test_no_call_before_the_entry_points_are_known():
    """In a process of its own: a call ahead of init, and an init without an entry point, are exceptions."""
    import subprocess
    import sys
    code = """
import torch
from paper_2603_14360_amd import _call
for call, error in ((lambda: _call.fwd(*[0] * 16), RuntimeError), (lambda: _call.bwd(*[0] * 26), RuntimeError),
                    (lambda: _call.init(None, 1), ValueError), (lambda: _call.init(1, 0), ValueError),
                    (lambda: _call.fwd(*[0] * 16), RuntimeError)):
    try:
        call()
    except error:
        continue
    raise SystemExit("no %s" % error)
"""
    assert subprocess.run([sys.executable, "-c", code], cwd=mb.os.path.dirname(mb._HERE)).returncode == 0
