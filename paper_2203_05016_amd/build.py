"""Build the C-ABI library (hipcc, gfx950 only) in-tree.

    python -m paper_2203_05016_amd.build
    python -m paper_2203_05016_amd.build --host-sanitized   # g++ ASan/UBSan build of the host-only sources

The results are ``paper_2203_05016_amd/libshflbw.so``, which links against the HIP
runtime only (no torch), and ``paper_2203_05016_amd/_torch_calls.so``, the binding's
native calls on torch tensors (host code, g++; left out where torch or its headers are missing).
"""
import contextlib
import os
import subprocess
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libshflbw.so")
SOURCES = ["compress.cpp", "pattern_search.cpp", "api_device.hip", "launch_gather_f16.hip", "launch_gather_bf16.hip",
           "launch_gather_conv_f16.hip", "launch_gather_conv_bf16.hip", "launch_gather_stride2_f16.hip", "launch_gather_stride2_bf16.hip",
           "launch_resident_f16.hip", "launch_resident_bf16.hip",
           "launch_resident_conv_f16.hip", "launch_resident_conv_bf16.hip", "layernorm_transpose.hip"]
# packed fp32 instructions are switched off for all device code
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wno-unused-command-line-argument",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]


TORCH_CALLS = os.path.join(HERE, "_torch_calls.so")


def _torch_calls_command(out):
    """The compiler's command line, or None without torch or the headers of torch or Python: the
    library needs neither, and the binding does without the native calls."""
    import sysconfig
    try:
        import torch
        from torch.utils import cpp_extension
    except ImportError:
        return None
    libdir = os.path.join(os.path.dirname(torch.__file__), "lib")
    includes = cpp_extension.include_paths() + [sysconfig.get_paths()["include"], os.path.join(ROOT, "include")]
    for header in ("ATen/core/Tensor.h", "Python.h"):
        if not any(os.path.exists(os.path.join(i, header)) for i in includes):
            return None
    return (["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch._C._GLIBCXX_USE_CXX11_ABI,
             "-DSHFLBW_TORCH_VERSION=\"%s\"" % torch.__version__,
             os.path.join(CSRC, "torch_calls.cpp"), "-o", out] + sum([["-isystem", i] for i in includes], []) +
            ["-L", libdir, "-ltorch_python", "-ltorch_cpu", "-ltorch", "-lc10"])


@contextlib.contextmanager
def _temporary(path):
    """A name beside path to build it under; what is still there afterwards (a step failed) is removed."""
    tmp = path + ".tmp.%d" % os.getpid()
    try:
        yield tmp
    finally:
        with contextlib.suppress(FileNotFoundError):
            os.remove(tmp)


def _run_all(jobs, verbose):
    """Runs the (name, command) jobs side by side; raises on a failure, when all have ended (none writes later)."""
    procs = [(name, subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)) for name, cmd in jobs]
    try:
        for name, p in procs:
            out = p.communicate()[0].decode()
            keep = [l for l in out.splitlines() if "packed-fp32-ops" not in l]
            if p.returncode != 0:
                sys.stderr.write(out)
                raise RuntimeError("compiler failed on %s" % name)
            if verbose and keep:
                print("\n".join(keep))
    finally:
        for _, p in procs:
            if p.returncode is None:
                p.communicate()


def build(verbose=True, extra=()):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objs, jobs = [], []
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    t0 = time.time()
    for src in SOURCES:
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        jobs.append((src, [hipcc, "-x", "hip", "-c", os.path.join(CSRC, src), "-o", obj] + FLAGS + list(extra)))
        objs.append(obj)
    with _temporary(LIB) as lib_tmp, _temporary(TORCH_CALLS) as calls_tmp:
        calls_command = _torch_calls_command(calls_tmp)
        if calls_command:
            jobs.append(("torch_calls.cpp", calls_command))
        _run_all(jobs, verbose)
        subprocess.check_call([hipcc, "-shared", "-fPIC", "--offload-arch=gfx950", "-o", lib_tmp] + objs)
        os.replace(lib_tmp, LIB)
        if calls_command:
            os.replace(calls_tmp, TORCH_CALLS)
    if not calls_command:
        if os.path.exists(TORCH_CALLS):   # of another torch
            os.remove(TORCH_CALLS)
        print("no torch or no headers: built without %s" % os.path.basename(TORCH_CALLS))
    if verbose:
        print("built %s in %.1f s" % (LIB, time.time() - t0))
    return LIB


HOST_SOURCES = ["compress.cpp", "pattern_search.cpp"]
HOST_SANITIZED_LIB = os.path.join(HERE, "_build", "libshflbw_host_sanitized.so")


def build_host_sanitized():
    """The host-only part of the library (offline compression, pattern search, the test
    hooks: no HIP call in it) compiled with g++ under AddressSanitizer and
    UndefinedBehaviorSanitizer, as a library of its own for the CPU tests.  Returns
    (path of the library, path of the sanitizer runtime to preload)."""
    os.makedirs(os.path.dirname(HOST_SANITIZED_LIB), exist_ok=True)
    with _temporary(HOST_SANITIZED_LIB) as tmp:
        subprocess.check_call(["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer",
                               "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined",
                               "-fPIC", "-shared", "-Wall", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                               "-o", tmp] + [os.path.join(CSRC, f) for f in HOST_SOURCES])
        os.replace(tmp, HOST_SANITIZED_LIB)
    runtime = subprocess.check_output(["g++", "-print-file-name=libasan.so"]).decode().strip()
    return HOST_SANITIZED_LIB, os.path.realpath(runtime)


if __name__ == "__main__":
    if sys.argv[1:] == ["--host-sanitized"]:
        print("built %s (preload %s)" % build_host_sanitized())
    else:
        build(extra=sys.argv[1:])
