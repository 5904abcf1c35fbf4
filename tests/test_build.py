"""The build removes what it had begun when a step fails: nothing but the finished files is ever left
beside the sources.  No GPU, and no real compiler run: stand-ins write their output and fail or succeed."""
import os
import stat
import subprocess

import pytest

from paper_2203_05016_amd import build as lib_build


def _tool(path, body):
    path.write_text("#!/bin/sh\n" + body)
    path.chmod(path.stat().st_mode | stat.S_IXUSR)
    return str(path)


WRITE_OUTPUT = 'while [ $# -gt 0 ]; do [ "$1" = -o ] && : > "$2"; shift; done\n'


@pytest.mark.parametrize("compile_ok,link_ok,calls_ok", [(False, True, True), (True, False, True), (True, True, False),
                                                         (True, True, True)])
def test_failed_build_leaves_no_temporary_files(monkeypatch, tmp_path, compile_ok, link_ok, calls_ok):
    out = tmp_path / "out"
    out.mkdir()
    monkeypatch.setattr(lib_build, "HERE", str(out))
    monkeypatch.setattr(lib_build, "LIB", str(out / "libshflbw.so"))
    monkeypatch.setattr(lib_build, "TORCH_CALLS", str(out / "_torch_calls.so"))
    hipcc = _tool(tmp_path / "hipcc", 'case " $* " in *" -c "*) code=%d;; *) code=%d;; esac\n%sexit $code\n'
                  % (not compile_ok, not link_ok, WRITE_OUTPUT))
    monkeypatch.setenv("HIPCC", hipcc)
    calls = _tool(tmp_path / "g++", WRITE_OUTPUT + "exit %d\n" % (not calls_ok))
    monkeypatch.setattr(lib_build, "_torch_calls_command", lambda o: [calls, "-o", o])
    ok = compile_ok and link_ok and calls_ok
    if ok:
        lib_build.build(verbose=False)
    else:
        with pytest.raises((RuntimeError, subprocess.CalledProcessError)):
            lib_build.build(verbose=False)
    assert sorted(os.listdir(out)) == ["_build"] + (["_torch_calls.so", "libshflbw.so"] if ok else [])


def test_temporary_names_are_ignored_by_git():
    names = [p + ".tmp.123" for p in (lib_build.LIB, lib_build.TORCH_CALLS, lib_build.HOST_SANITIZED_LIB)]
    r = subprocess.run(["git", "check-ignore"] + names, cwd=lib_build.ROOT, stdout=subprocess.PIPE, stderr=subprocess.PIPE)
    if r.returncode == 128:
        pytest.skip("not a git checkout")
    assert r.stdout.decode().split() == names
