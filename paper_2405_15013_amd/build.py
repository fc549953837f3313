"""Build libks.so (the HIP kernels and the C ABI) in place for gfx950.

    python -m paper_2405_15013_amd.build [--incremental]

Every HIP/C++ source under csrc/ is compiled with hipcc for gfx950 and linked
into paper_2405_15013_amd/libks.so; then bind/ks_torch.cpp, host code against
PyTorch's C++ headers, becomes the Python module _ks_torch (libks.so needs
neither; without the module the binding calls it by ctypes).  Packed-FP32 instruction selection is turned
off for device code (``-Xclang -target-feature -Xclang -packed-fp32-ops``); the
host pass warns that it does not know that feature, which is harmless.
"""
import concurrent.futures
import importlib.util
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libks.so")
BIND = os.path.join(HERE, "bind", "ks_torch.cpp")
BIND_LIB = os.path.join(HERE, "_ks_torch.so")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"

COMMON = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=" + ARCH,
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
    "-I" + os.path.join(HERE, "..", "include"),
]


def sources():
    return sorted(os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp")))


def _headers_mtime():
    hdrs = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith(".h")]
    inc = os.path.join(HERE, "..", "include")
    hdrs += [os.path.join(inc, f) for f in os.listdir(inc) if f.endswith(".h")]
    return max([os.path.getmtime(h) for h in hdrs] + [os.path.getmtime(__file__)])


def _compile(src, incremental=False):
    obj = os.path.join(BUILD, os.path.basename(src) + ".o")
    if incremental and os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), _headers_mtime()):
        return obj
    cmd = [HIPCC] + COMMON + ["-c", src, "-o", obj]
    r = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    err = "\n".join(l for l in (r.stdout + r.stderr).splitlines() if noise not in l)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s" % (" ".join(cmd), err))
    if err.strip():
        sys.stderr.write(err + "\n")
    return obj


def _bind_is_current():
    """_ks_torch is newer than its sources and was built for this PyTorch (its
    classes' layouts are compiled in)."""
    import torch
    if not os.path.exists(BIND_LIB) or os.path.getmtime(BIND_LIB) <= max(os.path.getmtime(BIND), _headers_mtime()):
        return False
    with open(BIND_LIB, "rb") as fh:
        return b"built for PyTorch %s;" % torch.__version__.encode() in fh.read()


def _build_bind(incremental=False):
    """The native form of the Python binding (no device code)."""
    import sysconfig

    import torch
    if incremental and _bind_is_current():
        return BIND_LIB
    root = os.path.dirname(torch.__file__)
    tmp = BIND_LIB + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           '-DKS_TORCH_VERSION="%s"' % torch.__version__,
           "-isystem", os.path.join(root, "include"),
           "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
           "-isystem", sysconfig.get_paths()["include"], BIND, "-o", tmp,
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError("compile failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))
    if r.stderr.strip():
        sys.stderr.write(r.stderr)
    os.replace(tmp, BIND_LIB)
    return BIND_LIB


def build(verbose=True, incremental=False):
    """Compile every source (or, with incremental=True, only those older than
    their object file or any header), link libks.so and build _ks_torch."""
    os.makedirs(BUILD, exist_ok=True)
    srcs = sources()
    torch_here = importlib.util.find_spec("torch") is not None
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(srcs) + 1)) as ex:
        bind = ex.submit(_build_bind, incremental) if torch_here else None
        objs = list(ex.map(lambda s: _compile(s, incremental), srcs))
        tmp = LIB + ".tmp%d" % os.getpid()
        cmd = [HIPCC, "-shared", "-fPIC", "--offload-arch=" + ARCH, "-o", tmp] + objs
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("link failed: %s\n%s%s" % (" ".join(cmd), r.stdout, r.stderr))
        os.replace(tmp, LIB)
        if verbose:
            print("built", LIB)
        # The module only once the library is there, which does not need it.
        if bind is None:
            sys.stderr.write("no PyTorch: _ks_torch not built\n")
        elif bind.result() and verbose:
            print("built", BIND_LIB)
    return LIB


if __name__ == "__main__":
    build(incremental="--incremental" in sys.argv[1:])
