"""The build's parts stand on their own: the C library does not wait for the Python module, and a part that is
missing says how to build it.  The compilers are stand-ins that write their output file."""
import os
import stat

import pytest
import torch

from paper_2603_06938_amd import binding as sw
from paper_2603_06938_amd import build as b


@pytest.fixture
def tree(tmp_path, monkeypatch):
    cc = tmp_path / "cc"
    cc.write_text('#!/bin/sh\nwhile [ $# -gt 1 ]; do [ "$1" = -o ] && : > "$2"; shift; done\n')
    cc.chmod(cc.stat().st_mode | stat.S_IEXEC)
    monkeypatch.setattr(b, "HIPCC", str(cc))
    monkeypatch.setattr(b, "OBJ", str(tmp_path / "_build"))
    monkeypatch.setattr(b, "LIB", str(tmp_path / "libswimba.so"))
    monkeypatch.setattr(b, "NATIVE", str(tmp_path / "_native.so"))
    return tmp_path


def test_the_library_is_linked_where_the_module_does_not_compile(tree, monkeypatch):
    def fail(verbose):
        raise RuntimeError("no torch headers")
    monkeypatch.setattr(b, "_compile_native", fail)
    with pytest.raises(RuntimeError, match="no torch headers"):      # and it is said
        b.build()
    assert os.path.exists(b.LIB) and not os.path.exists(b.NATIVE)


def test_the_library_builds_without_torch(tree, monkeypatch):
    find = b.importlib.util.find_spec
    monkeypatch.setattr(b.importlib.util, "find_spec", lambda n, *a: None if n == "torch" else find(n, *a))
    monkeypatch.setattr(b, "_compile_native", lambda verbose: pytest.fail("compiled against torch"))
    assert b.build() == b.LIB and os.path.exists(b.LIB)


def test_a_missing_module_says_what_to_run(tmp_path, monkeypatch):
    monkeypatch.setattr(sw, "_native", None)
    monkeypatch.setattr(sw, "NATIVE_PATH", str(tmp_path / "_native.so"))
    t = torch.zeros(1, 2, 3, 4)
    with pytest.raises(RuntimeError, match="not built.*g.build"):
        sw.swimba_router_linear(t, t)
