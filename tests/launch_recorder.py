"""What a scan call would launch, found on the CPU: the library runs in a process of its own whose
HIP runtime entry points are replaced by a recorder, so the dispatch, the sizing and every launch
argument are real and nothing is executed.

    launches([{"call": "fwd", "desc": {...}, "ws": address or None, "ws_bytes": n, ...}, ...])
        -> [{"rc": status, "launches": [{"kernel": name, "grid": n, "block": n, "partial": addr}]}]

`kernel` is the demangled name with its template arguments; `partial` is the address of the partial
sums of y that a forward kernel was given (None for other kernels).  `opts` and `ckpt` (truth
values) switch on the options of the layer and the checkpoint buffer."""
import ctypes
import json
import os
import re
import subprocess
import sys
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2603_14360_amd", "libm2rnn.so")

_STUB = r"""
#include <stdint.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_;
#define MOST 4096
static const void *fn_[MOST]; static const char *name_[MOST]; static int n_;
static struct { const char *name; unsigned grid[3], block; uint64_t partial; } rec_[MOST];
static int nrec_;
static dim3_ g_, b_; static size_t sh_; static void *st_;
void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterVar(void **m, void *v, char *h, char *d, int e, size_t s, int c, int g) {}
void __hipRegisterFunction(void **m, const void *fn, char *dev, const char *name, unsigned t,
                           void *a, void *b, void *c, void *d, int *w) {
  if (n_ < MOST) { fn_[n_] = fn; name_[n_++] = name; }
}
int __hipPushCallConfiguration(dim3_ g, dim3_ b, size_t sh, void *st) { g_ = g; b_ = b; sh_ = sh; st_ = st; return 0; }
int __hipPopCallConfiguration(dim3_ *g, dim3_ *b, size_t *sh, void **st) { *g = g_; *b = b_; *sh = sh_; *st = st_; return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
int hipGetSymbolAddress(void **p, const void *s) { *p = (void *)0x7000000; return 0; }
int hipLaunchKernel(const void *fn, dim3_ g, dim3_ b, void **args, size_t sh, void *st) {
  if (nrec_ == MOST) return 1;
  const char *name = "?";
  for (int i = 0; i < n_; ++i) if (fn_[i] == fn) name = name_[i];
  rec_[nrec_].name = name;
  rec_[nrec_].grid[0] = g.x; rec_[nrec_].grid[1] = g.y; rec_[nrec_].grid[2] = g.z;
  rec_[nrec_].block = b.x * b.y * b.z;
  rec_[nrec_].partial = ~0ull;
  if (strstr(name, "half_fwd_kernel") || strstr(name, "mfma_fwd_kernel") || strstr(name, "quad_fwd_kernel"))
    memcpy(&rec_[nrec_].partial, args[1], 8);
  ++nrec_;
  return 0;
}
int rec_count(void) { return nrec_; }
void rec_clear(void) { nrec_ = 0; }
const char *rec_name(int i) { return rec_[i].name; }
unsigned rec_num(int i, int w) { return w < 3 ? rec_[i].grid[w] : rec_[i].block; }
uint64_t rec_partial(int i) { return rec_[i].partial; }
int rec_kernels(void) { return n_; }
const char *rec_kernel(int i) { return name_[i]; }
"""


def _run(stub_path, request):
    """In the child: the recorder first and globally, so that the library binds to it."""
    stub = ctypes.CDLL(stub_path, mode=ctypes.RTLD_GLOBAL)
    stub.rec_name.restype = stub.rec_kernel.restype = ctypes.c_char_p
    stub.rec_num.restype = ctypes.c_uint
    stub.rec_partial.restype = ctypes.c_uint64
    sys.path.insert(0, ROOT)
    from paper_2603_14360_amd import binding as mb
    sys.modules.setdefault("torch", type(sys)("torch"))  # (the binding's loader only imports it)
    L = mb.lib()
    if request == "kernels":
        return [stub.rec_kernel(i).decode() for i in range(stub.rec_kernels())]
    A = ctypes.c_void_p(0x1000000)
    out = []
    for c in request:
        stub.rec_clear()
        desc = mb.make_desc(**c["desc"])
        V = ctypes.c_void_p
        ws, n = V(c["ws"]) if c.get("ws") else None, c.get("ws_bytes", 0)
        ck = A if c.get("ckpt") else None
        a = A.value
        o = mb.m2rnn_opts(a, a, 1.0, a, a, a, a) if c.get("opts") else mb.m2rnn_opts()
        if c["call"] == "fwd":
            rc = L.m2rnn_fwd_opt(desc, o, A, A, A, A, A, A, A, A, ck, ws, n, None)
        elif c["call"] == "static":
            rc = L.m2rnn_fwd_static(desc, o, A, A, A, A, A, A, A, A, ck, None)
        else:
            rc = L.m2rnn_bwd_opt(desc, o, A, A, A, A, A, A, ck, A, A, A, A, A, A, A, A, ws, n, None)
        rows = []
        for i in range(stub.rec_count()):
            p = stub.rec_partial(i)
            g = 1
            for w in range(3):
                g *= stub.rec_num(i, w)
            rows.append({"kernel": stub.rec_name(i).decode(), "grid": g, "block": stub.rec_num(i, 3),
                         "partial": None if p == 2 ** 64 - 1 else p})
        out.append({"rc": rc, "launches": rows})
    return out


def _demangle(names):
    text = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True,
                          check=True).stdout.splitlines()
    short = [re.sub(r"m2rnn::|\(anonymous namespace\)::|^void |\(.*$", "", re.sub(r"\(anonymous namespace\)", "", t))
             for t in text]
    return dict(zip(names, [s.lstrip(":").replace("::", "") for s in short]))


def _child(request):
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "rec.c"), os.path.join(d, "rec.so")
        with open(src, "w") as f:
            f.write(_STUB)
        subprocess.check_call(["gcc", "-shared", "-fPIC", "-w", "-o", so, src])
        p = subprocess.run([sys.executable, os.path.abspath(__file__), so], input=json.dumps(request),
                           capture_output=True, text=True)
        assert p.returncode == 0, p.stderr
        return json.loads(p.stdout)


def launches(calls):
    out = _child(calls)
    names = sorted({l["kernel"] for r in out for l in r["launches"]})
    short = _demangle(names) if names else {}
    for r in out:
        for l in r["launches"]:
            l["kernel"] = short[l["kernel"]]
    return out


def kernels():
    """Every kernel compiled into the library."""
    return sorted(set(_demangle(_child("kernels")).values()))


if __name__ == "__main__":
    json.dump(_run(sys.argv[1], json.load(sys.stdin)), sys.stdout)
