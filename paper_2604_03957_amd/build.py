"""Compile csrc/*.hip into csrc/libbwta.so for gfx950 with hipcc (cross-compiles without a GPU).

Each source is its own translation unit: the files are compiled side by side (up to 8 at a time)
into objects under csrc/_build/ and then linked; the Python binding's host part (csrc/_bwta_native.so)
is compiled beside them with g++.  Every call compiles everything again unless
`incremental=True` (a developer convenience: objects newer than their source and every header are
kept)."""
import concurrent.futures
import glob
import hashlib
import os
import shutil
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(CSRC, "_build")
LIB = os.path.join(CSRC, "libbwta.so")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "--offload-arch=gfx950", "-fPIC",
    # packed-fp32 VALU forms are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function", "-Wno-unknown-attributes",
]


BINDING_SRC = os.path.join(CSRC, "binding_native.cpp")
BINDING = os.path.join(CSRC, "_bwta_native.so")
BINDING_ID = os.path.join(OBJ, "binding_identity.txt")  # of the extension that is there, for the incremental build


def _binding_identity(bid):
    """What the extension must have been built for: these sources, this torch, this Python."""
    import torch
    return "%s %s %d.%d" % ((bid, torch.__version__) + sys.version_info[:2])


def _binding_compiler():
    """The host compiler for the extension: $CXX, else g++, else the clang++ that comes with hipcc; None if there is none."""
    if os.environ.get("CXX"):
        return os.environ["CXX"]
    return shutil.which("g++") or shutil.which("clang++", path="/opt/rocm/llvm/bin")


def _binding_headers():
    """The header folders of this Python and this torch, or None where their headers are not installed."""
    import torch
    py, tc = sysconfig.get_paths()["include"], os.path.join(os.path.dirname(torch.__file__), "include")
    there = os.path.exists(os.path.join(py, "Python.h")) and os.path.exists(os.path.join(tc, "torch", "csrc", "autograd", "python_variable.h"))
    return (py, tc) if there else None


def build_binding(bid, verbose=True):
    """The host-only extension that marshals the per-layer calls (binding_native.cpp), against this torch and Python.  It
    holds the C signatures of include/bwta.h and says what it was built from and for, which the binding compares with the
    library before it uses it.  Returns None where there is nothing to build it with: the binding's Python forms make the
    calls then, some 1 us slower each."""
    compiler, headers = _binding_compiler(), _binding_headers()
    if compiler is None or headers is None:
        print("_bwta_native.so is not built: %s; the calls are marshalled in Python"
              % ("no C++ compiler" if compiler is None else "no headers of Python or torch"), flush=True)
        for left in (BINDING, BINDING_ID):
            if os.path.exists(left):
                os.remove(left)
        return None
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = BINDING + ".tmp%d" % os.getpid()
    cmd = [compiler, "-O2", "-std=c++17", "-shared", "-fPIC", "-fvisibility=hidden", "-Wall",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, '-DBWTA_IDENTITY="%s"' % _binding_identity(bid), "-I" + headers[0],
           "-isystem", headers[1], "-isystem", os.path.join(headers[1], "torch", "csrc", "api", "include"),
           BINDING_SRC, "-o", tmp, "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.check_call(cmd)
    os.replace(tmp, BINDING)
    with open(BINDING_ID, "w") as f:
        f.write(_binding_identity(bid))
    return BINDING


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _headers():
    return glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(HERE, "..", "include", "*.h"))


def build_id():
    """Digest of every source and header the library and its binding are built from (and of the compiler flags)."""
    h = hashlib.sha1(" ".join(HIPCC_FLAGS).encode())
    for f in sorted(sources() + _headers() + [BINDING_SRC], key=os.path.basename):
        h.update(os.path.basename(f).encode())
        h.update(open(f, "rb").read())
    return h.hexdigest()[:12]


def build_library(verbose=True, extra_flags=(), incremental=False, jobs=8):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    os.makedirs(OBJ, exist_ok=True)
    bid = build_id()
    newest_header = max(os.path.getmtime(h) for h in _headers())
    todo, objs = [], []
    for src in sources():
        obj = os.path.join(OBJ, os.path.basename(src)[:-4] + ".o")
        objs.append(obj)
        fresh = (incremental and not extra_flags and os.path.exists(obj)
                 and os.path.getmtime(obj) > max(os.path.getmtime(src), newest_header))
        if not fresh or os.path.basename(src) == "bwta_api.hip":
            todo.append((src, obj))

    def compile_one(job):
        src, obj = job
        cmd = [hipcc] + HIPCC_FLAGS + list(extra_flags) + ["-c", src, "-o", obj]
        if os.path.basename(src) == "bwta_api.hip":  # the one file that records the digest: always rebuilt
            cmd.insert(-4, '-DBWTA_BUILD_ID="%s"' % bid)
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.check_call(cmd)

    stale = not (incremental and os.path.exists(BINDING) and os.path.exists(BINDING_ID) and open(BINDING_ID).read() == _binding_identity(bid))
    with concurrent.futures.ThreadPoolExecutor(max_workers=max(1, min(jobs, len(todo) + 1))) as pool:
        binding = pool.submit(build_binding, bid, verbose) if stale else None
        list(pool.map(compile_one, todo))
        if binding:
            binding.result()
    tmp = LIB + ".tmp%d" % os.getpid()
    link = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    if verbose:
        print(" ".join(link), flush=True)
    subprocess.check_call(link)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    flags = [a for a in sys.argv[1:] if a != "--incremental"]
    build_library(extra_flags=flags, incremental="--incremental" in sys.argv[1:])
