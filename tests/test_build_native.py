"""The extension with the binding's native calls is made beside the library and is no condition for it: a package without
it takes every call through the Python forms, a build without a C compiler leaves a library and no extension (least of
all an old one), and where only the extension is missing only the extension is made."""
import os
import shutil
import stat
import subprocess
import sys

import pytest

from paper_2511_12653_amd import build

PACKAGE = os.path.dirname(os.path.abspath(build.__file__))

WITHOUT = r"""
import ctypes, inspect
from paper_2511_12653_amd import binding as fq
from paper_2511_12653_amd import fq_forward, fq_distill_loss
assert fq._fqcall is None and fq.library_path().startswith(%r)
t = fq.FqTensor(3, 5, 70000, fq.FQ_F16, -8, 7, 0.0, fq.FLT_MIN, 1.0, 0, 4096, 4096, None, 4096, None, 4096, 4096)
assert fq.fq_workspace_bytes(t, 2) == fq.fq_workspace_bytes([t], 2) > 0
fq._current_stream = lambda: 0
for call, args, status in ((fq.fq_forward, (fq.FqTensor(1, 1, 8, 7, -8, 7),), -2), (fq.fq_backward, (t, None), -6),
                           (fq.fq_plan_run, (ctypes.c_void_p(),), -1), (fq.fq_plan_run_adam, (ctypes.c_void_p(), 3), -1)):
    try:
        call(*args)
    except fq.FqError as e:
        assert e.status == status, (call, e.status)
    else:
        raise AssertionError(call)
assert str(inspect.signature(fq.fq_plan_run_adam)) == "(plan, step, stream=None)"
print("served")
"""


def test_a_package_without_the_extension_serves(tmp_path):
    there = tmp_path / "paper_2511_12653_amd"
    there.mkdir()
    for f in os.listdir(PACKAGE):
        if f.endswith(".py") or f == "libfq.so":
            shutil.copy(os.path.join(PACKAGE, f), str(there / f))
    p = subprocess.run([sys.executable, "-c", WITHOUT % str(tmp_path)], cwd=str(tmp_path), stdout=subprocess.PIPE,
                       stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0 and "served" in p.stdout, p.stdout


def _script(path, text):
    path.write_text("#!/bin/sh\n" + text)
    path.chmod(path.stat().st_mode | stat.S_IXUSR)
    return str(path)


@pytest.fixture
def elsewhere(tmp_path, monkeypatch):
    """build.py's outputs in a folder of their own, and stand-ins for both compilers (the last argument is the file)."""
    log = tmp_path / "log"
    say = "echo %%s >> %s; for a; do out=$a; done; echo %%s > \"$out\"" % log
    out = tmp_path / "out"
    out.mkdir()
    monkeypatch.setattr(build, "LIB", str(out / "libfq.so"))
    monkeypatch.setattr(build, "CALL", str(out / "_fqcall.so"))
    monkeypatch.setattr(build, "HIPCC", _script(tmp_path / "hipcc", say % ("hipcc", "library")))
    monkeypatch.setattr(build, "CC", _script(tmp_path / "cc", say % ("cc", "extension")) + " -pthread")
    return out, log


def test_both_files_appear_together(elsewhere):
    out, log = elsewhere
    assert build.ensure_built() == build.LIB and log.read_text().split() == ["hipcc", "cc"]
    assert sorted(os.listdir(out)) == ["_fqcall.so", "libfq.so"]


@pytest.mark.parametrize("compiler", ["false", "/nonexistent/cc"])
def test_no_compiler_leaves_the_library_alone_and_no_old_extension(elsewhere, monkeypatch, capsys, compiler):
    out, log = elsewhere
    (out / "libfq.so").write_text("old")
    (out / "_fqcall.so").write_text("old")
    monkeypatch.setattr(build, "CC", compiler)
    assert build.build() == build.LIB
    assert os.listdir(out) == ["libfq.so"] and (out / "libfq.so").read_text() == "library\n"
    assert "no native calls" in capsys.readouterr().err
    assert build.ensure_built() == build.LIB and os.listdir(out) == ["libfq.so"]


def test_a_failing_library_changes_nothing(elsewhere, monkeypatch):
    out, log = elsewhere
    (out / "libfq.so").write_text("old")
    (out / "_fqcall.so").write_text("old")
    monkeypatch.setattr(build, "HIPCC", "false")
    with pytest.raises(subprocess.CalledProcessError):
        build.build()
    assert sorted(os.listdir(out)) == ["_fqcall.so", "libfq.so"]
    assert (out / "libfq.so").read_text() == (out / "_fqcall.so").read_text() == "old"


def test_only_the_missing_extension_is_made(elsewhere):
    out, log = elsewhere
    (out / "libfq.so").write_text("old")
    build.ensure_built()
    assert log.read_text().split() == ["cc"] and sorted(os.listdir(out)) == ["_fqcall.so", "libfq.so"]
    assert (out / "libfq.so").read_text() == "old"
