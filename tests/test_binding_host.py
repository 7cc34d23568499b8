"""The native binding calls the library's entry points by address: it is built with the library, refused where it was compiled against another wk.h, and not
taken for absent where it does not load."""
import importlib.util
import os
import shutil
import sys
import types

import pytest

import paper_2605_22718_amd as wk
from paper_2605_22718_amd import build

PACKAGE = os.path.dirname(os.path.abspath(wk.__file__))


def test_build_makes_the_library_and_the_binding(monkeypatch):
    outputs = []
    monkeypatch.setattr(build, "_compile", lambda src: src + ".o")
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: outputs.append(cmd[cmd.index("-o") + 1]))
    build.build(force=True)
    assert set(outputs) == {build.LIB, build.BINDING}


def test_an_old_binding_is_built_again(monkeypatch):
    outputs = []
    monkeypatch.setattr(build, "_compile", lambda src: src + ".o")
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **kw: outputs.append(cmd[cmd.index("-o") + 1]))
    monkeypatch.setattr(build, "_is_newer", lambda product, deps: product != build.BINDING)
    build.build(force=False)
    assert outputs == [build.BINDING]


def test_library_and_binding_are_of_this_interface():
    assert isinstance(wk._native, types.ModuleType)
    assert build.interface_flag() == f"-DWK_INTERFACE=0x{wk._native.interface():016x}ull"
    assert wk.lib().wk_internal_interface() == wk._native.interface()


@pytest.mark.parametrize("says", [True, False])   # (one from before a binding said what it is of does not)
def test_a_binding_of_another_interface_is_refused(says, monkeypatch):
    def bind(*args):
        raise AssertionError("bound")
    other = wk.lib().wk_internal_interface() ^ 1
    monkeypatch.setattr(wk, "_lib", None)
    monkeypatch.setattr(wk, "_native", types.SimpleNamespace(bind=bind, **({"interface": lambda: other} if says else {})))
    with pytest.raises(ImportError, match="another include/wk.h"):
        wk.lib()
    assert wk._lib is None


@pytest.mark.parametrize("binding", [None, b"no library"])
def test_a_binding_that_does_not_load_is_not_taken_for_none(binding, tmp_path):
    shutil.copy(os.path.join(PACKAGE, "__init__.py"), tmp_path)
    os.symlink(os.path.join(PACKAGE, "libwk.so"), tmp_path / "libwk.so")
    if binding is not None:
        (tmp_path / "wk_binding.so").write_bytes(binding)
    spec = importlib.util.spec_from_file_location("wk_copy", tmp_path / "__init__.py", submodule_search_locations=[str(tmp_path)])
    copy = importlib.util.module_from_spec(spec)
    sys.modules["wk_copy"] = copy
    try:
        spec.loader.exec_module(copy)   # (to be built, the package has to be importable)
        if binding is None:
            assert copy.status_string(0) == "ok"
        else:
            with pytest.raises(ImportError, match="does not load"):
                copy.lib()
    finally:
        del sys.modules["wk_copy"]
