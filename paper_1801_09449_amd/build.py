"""Compile the gfx950 library (csrc/*.hip -> paper_1801_09449_amd/libtern.so) with hipcc, and the
binding's per-call path (csrc/tern_torch.cpp -> _tern_torch.so, host code only) with g++.

hipcc cross-compiles without a GPU present.  The library is built in-tree so that it travels with
the source tree; it is not installed anywhere.  Every call recompiles every source (one hipcc
process per file, side by side) and links the objects.
"""
import glob
import os
import shutil
import subprocess
import sys
import sysconfig
import tempfile
import warnings
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libtern.so")
NATIVE = os.path.join(HERE, "_tern_torch.so")

FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument",
    "-I", os.path.join(ROOT, "include"), "-I", CSRC,
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def _run(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    # the host pass warns that it does not know the packed-fp32 target feature: harmless
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        raise RuntimeError(cmd[0] + " failed:\n" + " ".join(cmd) + "\n" + out)
    if verbose and out.strip():
        print(out, flush=True)


def _native_lacks():
    """What is not there for compiling the torch side of the binding, or None."""
    if shutil.which("g++") is None:
        return "g++"
    if not os.path.exists(os.path.join(sysconfig.get_paths()["include"], "Python.h")):
        return "Python.h"
    try:
        from torch.utils import cpp_extension
        paths = cpp_extension.include_paths()
    except Exception as e:                      # torch itself, or something that its build tools import
        return "torch (%s)" % e
    if not any(os.path.exists(os.path.join(p, "torch", "csrc", "autograd", "python_variable.h")) for p in paths):
        return "torch's headers"
    return None


def _build_native(verbose):
    """The torch side of the binding, linked against libtern.so beside it.  Where its tools are missing there
    is no such file afterwards (the binding then makes its calls through ctypes); a source that does not
    compile is an error."""
    lacks = _native_lacks()
    if lacks:
        if os.path.exists(NATIVE):
            os.remove(NATIVE)                   # of another build
        warnings.warn("_tern_torch.so is not built, %s is missing: calls take some microseconds more" % lacks)
        return
    from torch.utils import cpp_extension
    tmp = NATIVE + ".tmp.%d" % os.getpid()
    libs = cpp_extension.library_paths()
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden", "-I", os.path.join(ROOT, "include")]
    for p in cpp_extension.include_paths() + [sysconfig.get_paths()["include"]]:
        cmd += ["-isystem", p]
    cmd += ["-o", tmp, os.path.join(CSRC, "tern_torch.cpp"), "-L", HERE, "-l:libtern.so"]
    for p in libs:
        cmd += ["-L", p]
    cmd += ["-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10", "-Wl,-rpath,$ORIGIN"]
    try:
        _run(cmd, verbose)
        os.replace(tmp, NATIVE)
    finally:
        if os.path.exists(tmp):
            os.remove(tmp)


def build(verbose: bool = False, jobs: int = 0) -> str:
    """Always recompiles (under a minute with a few cores)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    jobs = jobs or min(8, os.cpu_count() or 1)
    tmpdir = tempfile.mkdtemp(prefix="tern_build_")
    try:
        objs = [os.path.join(tmpdir, os.path.basename(s)[:-4] + ".o") for s in sources()]
        with ThreadPoolExecutor(max_workers=jobs) as pool:
            list(pool.map(lambda so: _run([hipcc] + FLAGS + ["-c", so[0], "-o", so[1]], verbose),
                          zip(sources(), objs)))
        tmp = LIB + ".tmp.%d" % os.getpid()
        try:
            _run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs, verbose)
            os.replace(tmp, LIB)
        finally:
            if os.path.exists(tmp):
                os.remove(tmp)
        _build_native(verbose)
    finally:
        shutil.rmtree(tmpdir, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-q" not in sys.argv))
