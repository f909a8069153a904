"""The package with and without the binding's extension module: _fast.so marshals
calls, and libtri.so, which holds everything else, needs neither it nor torch."""
import importlib.util
import os
import shutil
import subprocess
import sys

import torch

from tests.conftest import ROOT

PKG = "paper_2609_37241_amd"
PROBE = f"""
import warnings
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    import {PKG} as tri
print(tri._native is not None, [str(w.message) for w in seen if w.category is RuntimeWarning])
f = tri.SpecCache._fast
print([getattr(f, n)(1, 2) for n in ("rmsnorm", "residual_rmsnorm", "swiglu", "silu", "add",
       "masked_fill", "embedding", "rope", "chain", "layers")], f.close())
"""


def _package(tmp_path, fast):
    """A copy of the package whose _fast.so is `fast` (bytes), or absent."""
    src, dst = os.path.join(ROOT, PKG), tmp_path / PKG
    dst.mkdir()
    for f in os.listdir(src):
        if f.endswith(".py") or f == "libtri.so":
            shutil.copy(os.path.join(src, f), dst / f)
    if fast is not None:
        (dst / "_fast.so").write_bytes(fast)
    r = subprocess.run([sys.executable, "-c", PROBE], cwd=tmp_path, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return r.stdout.strip().split("\n")


def _built():
    with open(os.path.join(ROOT, PKG, "_fast.so"), "rb") as f:
        return f.read()


def test_the_built_module_is_used(tmp_path):
    assert _package(tmp_path, _built())[0] == "True []"


def test_imports_without_the_extension_module(tmp_path):
    for i, fast in enumerate((None, b"not a library")):
        d = tmp_path / str(i)
        d.mkdir()
        state, calls = _package(d, fast)
        assert state.startswith("False") and "_fast.so is not used" in state
        assert calls == str([None] * 10) + " None"


def test_a_module_built_against_another_torch_is_not_used(tmp_path):
    version = torch.__version__.encode()
    assert version in _built()
    other = _built().replace(version, bytes([version[0] + 1]) + version[1:])
    state = _package(tmp_path, other)[0]
    assert state.startswith("False") and "built against torch" in state


def test_libtri_builds_without_torch(tmp_path, monkeypatch):
    """The same commands as ever for libtri.so, none for the extension module."""
    spec = importlib.util.spec_from_file_location("_tri_build", os.path.join(ROOT, PKG, "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    find = importlib.util.find_spec
    monkeypatch.setattr(importlib.util, "find_spec", lambda n, *a: None if n == "torch" else find(n, *a))
    for name in ("BUILD", "LIB", "FAST_LIB", "BENCH_LIB", "HOSTCOST_LIB", "JIT_PRELUDE"):
        monkeypatch.setattr(build, name, str(tmp_path / os.path.basename(getattr(build, name))))
    cmds = []

    def run(cmd):
        cmds.append(cmd)
        with open(cmd[cmd.index("-o") + 1], "wb"):
            pass

    monkeypatch.setattr(build, "_run", run)
    assert build.build() == build.LIB and os.path.exists(build.LIB)
    assert not os.path.exists(build.FAST_LIB) and os.path.exists(build.HOSTCOST_LIB)
    assert not any("fast.cpp" in a for c in cmds for a in c)
