"""Builds the HIP library in-tree with hipcc for gfx950 (cross-compiles without a GPU) and the binding's tensor check with g++."""
import glob
import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libserveflow_hip.so")
MARSHAL_SRC = os.path.join(CSRC, "marshal.cpp")

# -ffp-contract=off: the feature statistics are defined with one rounding per operation.
# The packed-fp32 feature is switched off for device code (hipcc's host pass does not know
# the feature and says so; that warning is harmless).
# Sums of MFMAs stay in ordinary vector registers: the epilogues work on them, and a copy out of an accumulation
# register costs an instruction each.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-mllvm", "-amdgpu-mfma-vgpr-form=1",
    "-Wall", "-Wno-unused-function",
]


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")))


def marshal_path() -> str:
    """Where the tensor check for this Python and torch is, or would be: it holds for no other."""
    import torch
    return os.path.join(HERE, "_marshal.%s.torch-%s.so" % (sys.implementation.cache_tag, torch.__version__))


def is_stale() -> bool:
    marshal = marshal_path()
    if not os.path.exists(LIB) or not os.path.exists(marshal) or os.path.getmtime(MARSHAL_SRC) > os.path.getmtime(marshal):
        return True
    t = os.path.getmtime(LIB)
    deps = sources() + glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(ROOT, "include", "*.h"))
    return any(os.path.getmtime(p) > t for p in deps)


def build_marshal() -> str:
    """Compile the tensor check (csrc/marshal.cpp) against the installed torch; returns its path."""
    import torch
    from torch.utils import cpp_extension
    path = marshal_path()
    tmp = path + ".tmp.%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-fvisibility=hidden",
           "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI, "-I" + sysconfig.get_paths()["include"],
           *["-I" + p for p in cpp_extension.include_paths()], MARSHAL_SRC, "-o", tmp,
           *["-L" + p for p in cpp_extension.library_paths()], "-ltorch_python", "-ltorch_cpu", "-lc10"]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("%s failed:\n%s" % (cmd[0], res.stdout))
    os.replace(tmp, path)
    return path


def build(force: bool = True, verbose: bool = False) -> str:
    """Compile every kernel file into one shared library, and the tensor check; returns the library's path."""
    if not force and not is_stale():
        return LIB
    build_marshal()
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp.%d" % os.getpid()
    cmd = [hipcc, *HIPCC_FLAGS, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, *sources(), "-o", tmp]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    out = "\n".join(l for l in res.stdout.splitlines() if "packed-fp32-ops" not in l)
    if res.returncode != 0:
        if os.path.exists(tmp):
            os.remove(tmp)
        raise RuntimeError("hipcc failed:\n" + out)
    if verbose and out.strip():
        print(out)
    os.replace(tmp, LIB)
    return LIB


SAN_LIB = os.path.join(ROOT, "_build", "libserveflow_hip_hostsan.so")
CLANG_ASAN_RUNTIME = "/opt/rocm/llvm/lib/clang"


def build_host_sanitized() -> str:
    """A second copy of the library whose HOST code (argument checks, the threshold algorithms, workspace
    arithmetic) is instrumented with AddressSanitizer and UndefinedBehaviorSanitizer; the device code is
    built as always.  For CPU-side tests only: load it with the sanitizer runtime preloaded
    (asan_runtime()) and SERVEFLOW_LIB pointing at it."""
    os.makedirs(os.path.dirname(SAN_LIB), exist_ok=True)
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = [f for f in HIPCC_FLAGS if f != "-O3"] + [
        "-O1", "-g", "-Xarch_host", "-fsanitize=address", "-Xarch_host", "-fsanitize=undefined",
        "-Xarch_host", "-fno-sanitize-recover=undefined", "-shared-libsan"]
    cmd = [hipcc, *flags, "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, *sources(), "-o", SAN_LIB]
    res = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if res.returncode != 0:
        raise RuntimeError("hipcc (host sanitizers) failed:\n" + res.stdout)
    return SAN_LIB


def asan_runtime() -> str:
    """Path of the AddressSanitizer runtime that matches hipcc's host compiler."""
    hits = glob.glob(os.path.join(CLANG_ASAN_RUNTIME, "*", "lib", "linux", "libclang_rt.asan-x86_64.so"))
    if not hits:
        raise RuntimeError("no libclang_rt.asan-x86_64.so under " + CLANG_ASAN_RUNTIME)
    return sorted(hits)[-1]


if __name__ == "__main__":
    print(build(force=True, verbose=True))
