"""Builds libm2rnn.so (the C-ABI library) in-tree with hipcc for gfx950, and _call, the host-only Python
module that the binding calls it with (for the Python and the torch that build it: the file name says
the one, the module the other).

    python -m paper_2603_14360_amd.build

Every .hip file under csrc/ is compiled to an object (in parallel) and linked
into ``paper_2603_14360_amd/libm2rnn.so``.  Packed-FP32 instruction selection
is switched off for device code.
"""
import concurrent.futures
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libm2rnn.so")
CALL = os.path.join(HERE, "_call" + sysconfig.get_config_var("EXT_SUFFIX"))

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CXX = os.environ.get("CXX", "g++")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-command-line-argument",
]


def _compile(src):
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in proc.stderr.splitlines() if noise not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _compile_call():
    """csrc/py_call.cpp against the headers of the torch that is installed."""
    import torch
    root = os.path.dirname(torch.__file__)
    inc = [os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
           sysconfig.get_paths()["include"]]
    tmp = CALL + ".tmp%d" % os.getpid()
    cmd = [CXX, "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
           '-DM2RNN_TORCH_VERSION="%s"' % torch.__version__] + ["-I" + i for i in inc]
    cmd += [os.path.join(CSRC, "py_call.cpp"), "-o", tmp, "-L" + os.path.join(root, "lib"),
            "-ltorch_python", "-ltorch_cpu", "-lc10"]
    try:
        proc = subprocess.run(cmd, capture_output=True, text=True)
    except OSError as e:
        raise RuntimeError("%s, for py_call.cpp: %s" % (CXX, e)) from e
    if proc.returncode != 0:
        raise RuntimeError("%s failed on py_call.cpp:\n%s" % (CXX, proc.stderr))
    os.replace(tmp, CALL)
    untagged = os.path.join(HERE, "_call.so")  # (one that any Python would take for its own)
    if os.path.exists(untagged) and untagged != CALL:
        os.remove(untagged)


def build(verbose=True):
    os.makedirs(OBJ, exist_ok=True)
    sources = sorted(glob.glob(os.path.join(CSRC, "*.hip")))
    if not sources:
        raise RuntimeError("no HIP sources under " + CSRC)
    with concurrent.futures.ThreadPoolExecutor(max_workers=8) as pool:
        objs = list(pool.map(_compile, sources))
    tmp = LIB + ".tmp%d" % os.getpid()
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    # (behind the library, which needs neither torch nor a host compiler)
    try:
        import torch  # noqa: F401
    except ImportError:
        print("torch is not installed: %s, which binding.Scan calls the library with, is not built" % CALL)
        return LIB
    _compile_call()
    return LIB


if __name__ == "__main__":
    build()
