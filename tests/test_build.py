"""The library is built from the sources that are there: all of them compile, and no other library is taken for theirs."""
import os
import shutil
import subprocess
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_1904_01038_amd import build

needs_hipcc = pytest.mark.skipif(shutil.which("hipcc") is None, reason="no hipcc")


@needs_hipcc
def test_every_source_compiles():
    def errors(source):
        r = subprocess.run(["hipcc", *build.FLAGS, "-fsyntax-only", os.path.join(build.CSRC, source)], capture_output=True, text=True)
        return [] if r.returncode == 0 else [source] + [l for l in r.stderr.splitlines() if "error:" in l]
    with ThreadPoolExecutor(max_workers=8) as ex:
        found = [e for e in ex.map(errors, build.SOURCES) if e]
    assert not found, found


@needs_hipcc
def test_a_build_that_fails_leaves_no_library(tmp_path, monkeypatch):
    csrc, lib = tmp_path / "csrc", tmp_path / "libtfm.so"
    csrc.mkdir()
    (csrc / "a.hip").write_text("int a() { return undeclared; }\n")
    lib.write_bytes(b"of an earlier build")
    for name, value in [("CSRC", csrc), ("LIB", lib), ("OBJ", tmp_path / "_build")]:
        monkeypatch.setattr(build, name, str(value))
    monkeypatch.setattr(build, "SOURCES", ["a.hip"])
    with pytest.raises(RuntimeError, match="undeclared"):
        build.build(verbose=False)
    assert not lib.exists()


@pytest.mark.parametrize("changed", ["tfm.hip", "kernels.h"])
def test_a_library_of_other_sources_is_refused(tmp_path, monkeypatch, changed):
    import paper_1904_01038_amd as T
    from paper_1904_01038_amd import binding
    if not os.path.exists(T.lib_path()):
        build.build(verbose=False)
    monkeypatch.setattr(binding, "_lib", None)
    T.lib()                                   # (of the sources as they are)
    shutil.copytree(build.CSRC, tmp_path / "csrc")
    monkeypatch.setattr(build, "CSRC", str(tmp_path / "csrc"))
    monkeypatch.setattr(binding, "_lib", None)
    T.lib()                                   # (elsewhere, but the same)
    with open(tmp_path / "csrc" / changed, "a") as f:
        f.write("// one more line\n")
    monkeypatch.setattr(binding, "_lib", None)
    with pytest.raises(RuntimeError, match="other sources"):
        T.lib()
