"""The entry points have C linkage: when a host allocation fails, whatever they have to report, they
return a status, and no C++ exception leaves them.  A small program that fails every allocation during
the calls (tests/alloc_failure.cpp), run against the built library.  No GPU: every call is refused
before it reaches the device."""
import os
import subprocess

from paper_2203_05016_amd import binding, build as lib_build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_no_exception_leaves_an_entry_point(tmp_path):
    binding.lib()   # built
    exe = str(tmp_path / "alloc_failure")
    libdir = os.path.dirname(binding.LIB_PATH)
    rocm = "/opt/rocm/lib"
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(lib_build.ROOT, "include"), "-o", exe,
                           os.path.join(HERE, "alloc_failure.cpp"), binding.LIB_PATH, "-Wl,--allow-shlib-undefined",
                           "-Wl,-rpath," + libdir, "-Wl,-rpath," + rocm])
    r = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.PIPE, timeout=120,
                       env=dict(os.environ, LD_LIBRARY_PATH=rocm + ":" + os.environ.get("LD_LIBRARY_PATH", "")))
    assert r.returncode == 0, r.stdout.decode() + r.stderr.decode()
