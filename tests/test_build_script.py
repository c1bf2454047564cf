"""build.py with a stand-in compiler: both libraries are replaced together when
both compile, and a failure leaves the old ones and no temporary files."""
import importlib.util
import os
import stat
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture
def script(tmp_path, monkeypatch):
    """The build module writing to tmp_path; fake(name) makes hipcc fail for that
    library after writing a part of its output."""
    spec = importlib.util.spec_from_file_location(
        "build_under_test", os.path.join(ROOT, "paper_1504_01380_amd", "build.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    mod.LIB, mod.LIB_COUNT = str(tmp_path / "libswept.so"), str(tmp_path / "libswept_count.so")
    for lib in (mod.LIB, mod.LIB_COUNT):
        with open(lib, "w") as fh:
            fh.write("old")
    bindir = tmp_path / "bin"
    bindir.mkdir()

    def fake(fails=""):
        hipcc = bindir / "hipcc"
        hipcc.write_text('#!/bin/sh\nwhile [ "$1" != -o ]; do shift; done\nprintf new > "$2"\n'
                         'case "$2" in %s) exit 1;; esac\n' % (fails or "none"))
        hipcc.chmod(hipcc.stat().st_mode | stat.S_IXUSR)

    monkeypatch.setenv("PATH", "%s:%s" % (bindir, os.environ["PATH"]))
    return mod, fake, tmp_path


def contents(mod):
    return [open(p).read() for p in (mod.LIB, mod.LIB_COUNT)]


def test_both_are_replaced(script):
    mod, fake, d = script
    fake()
    assert mod.build() == mod.LIB
    assert contents(mod) == ["new", "new"] and len(os.listdir(d)) == 3


@pytest.mark.parametrize("fails", ["*libswept.so.tmp*", "*libswept_count.so.tmp*", "*"])
def test_a_failure_leaves_no_files_behind(script, fails):
    mod, fake, d = script
    fake(fails)
    with pytest.raises(subprocess.CalledProcessError):
        mod.build()
    assert contents(mod) == ["old", "old"]
    assert sorted(os.listdir(d)) == ["bin", "libswept.so", "libswept_count.so"]
