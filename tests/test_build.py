"""The library is built from the sources that are there: all of them compile."""
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
