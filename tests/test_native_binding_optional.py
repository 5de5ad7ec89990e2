"""_zq_host.so is a faster way to the same library, not a requirement: without it the library loads, with a warning, and the build
succeeds, where g++, Python's headers or a ROCm torch are missing."""
import os
import subprocess
import sys

import pytest

from paper_2206_01861_amd import build as zq_build

CODE = """
import sys, warnings
import paper_2206_01861_amd as zq
from paper_2206_01861_amd import binding
%s
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    zq.lib()
assert binding._host is None and zq.version() >= 100 and zq.gemm_schedule(1, 2048, 2048) is not None
assert any("_zq_host" in str(w.message) for w in seen), seen
"""


@pytest.mark.parametrize("missing", [
    "binding._HOST_PATH = '/nonexistent/_zq_host.so'",                                                       # not built
    "binding._HOST_PATH = sys.executable; sys.modules['paper_2206_01861_amd._zq_host'] = None",               # built, does not load
])
def test_library_loads_without_the_native_module(missing):
    r = subprocess.run([sys.executable, "-c", CODE % missing], capture_output=True, text=True, cwd=os.path.dirname(zq_build.HERE))
    assert r.returncode == 0, r.stderr


def test_build_goes_on_without_a_compiler_for_it(tmp_path, monkeypatch, capsys):
    old = tmp_path / "_zq_host.so"
    old.write_bytes(b"an older build")
    monkeypatch.setattr(zq_build, "HOST", str(old))
    monkeypatch.setenv("CXX", "/nonexistent/g++")
    assert zq_build._try_host() is False
    assert not old.exists() and "ctypes" in capsys.readouterr().err
