"""The binding without its native form, and when that counts as built (no GPU needed)."""
import os
import sys
import types

import pytest

from paper_2504_12285_amd import binding as bl
from paper_2504_12285_amd import build as hip_build

torch = pytest.importorskip("torch")


def test_without_the_native_form_calls_run_in_python(monkeypatch):
    import paper_2504_12285_amd as pkg
    monkeypatch.setattr(bl, "_native", None)
    monkeypatch.delattr(pkg, "_bl_torch", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2504_12285_amd._bl_torch", None)      # import raises ImportError
    with pytest.warns(RuntimeWarning, match="run in Python"):
        native = bl._first_native()
    assert bl._native is native
    for call in (native.quant, native.product, native.decode, native.run):
        assert call(1, 2, 3) is NotImplemented
    with pytest.raises(AssertionError):                                           # the Python form's own check
        bl.bl_quant_act_int8(torch.zeros((1, 64), dtype=torch.bfloat16))


def test_a_native_form_of_another_torch_is_not_used(monkeypatch):
    import paper_2504_12285_amd as pkg
    other = types.ModuleType("paper_2504_12285_amd._bl_torch", "built for torch 0.0.1")
    other.bind = lambda *a: pytest.fail("bound")
    monkeypatch.setattr(bl, "_native", None)
    monkeypatch.setattr(pkg, "_bl_torch", other, raising=False)
    monkeypatch.setitem(sys.modules, other.__name__, other)
    with pytest.warns(RuntimeWarning, match="torch 0.0.1"):
        assert isinstance(bl._first_native(), bl._PythonForm)


@pytest.fixture
def tree(tmp_path, monkeypatch):
    """A package folder whose library and extension are up to date."""
    for name in ("csrc", "include"):
        os.mkdir(str(tmp_path / name))
    paths = {"LIB_PATH": "lib.so", "TORCH_EXT_PATH": "_bl_torch.x.so", "TORCH_EXT_SOURCE": "csrc/bl_torch.cpp"}
    for name, f in paths.items():
        monkeypatch.setattr(hip_build, name, str(tmp_path / f))
    for name, f in (("PKG_DIR", ""), ("CSRC", "csrc"), ("INCLUDE", "include")):
        monkeypatch.setattr(hip_build, name, str(tmp_path / f))
    monkeypatch.setattr(hip_build, "SOURCES", ["a.hip"])
    for f in ("csrc/a.hip", "csrc/a.h", "csrc/bl_torch.cpp", "include/bitlinear.h"):
        (tmp_path / f).write_text("")
        os.utime(str(tmp_path / f), (1000, 1000))
    (tmp_path / "lib.so").write_text("old")
    (tmp_path / "_bl_torch.x.so").write_bytes(b"..." + hip_build._torch_mark() + b"...")
    return tmp_path


def test_what_makes_the_build_stale(tree, monkeypatch):
    assert not hip_build.is_stale()
    for f in ("csrc/a.hip", "csrc/a.h", "csrc/bl_torch.cpp", "include/bitlinear.h"):
        os.utime(str(tree / f), (1e10, 1e10))
        assert hip_build.is_stale(), f
        os.utime(str(tree / f), (1000, 1000))
    os.utime(str(tree / "include" / "bitlinear.h"), (1e10, 1e10))
    os.utime(str(tree / "lib.so"), (2e10, 2e10))                     # the library is newer than the header, the extension is not
    assert hip_build.is_stale()
    os.utime(str(tree / "include" / "bitlinear.h"), (1000, 1000))
    with monkeypatch.context() as m:
        m.setattr(hip_build, "torch_version", lambda: "0.0.1")
        assert hip_build.is_stale()
    os.remove(str(tree / "_bl_torch.x.so"))
    assert hip_build.is_stale()
    monkeypatch.setattr(hip_build, "torch_ext_missing", lambda: "no g++")
    assert not hip_build.is_stale()                                  # nothing that could be built is missing


@pytest.mark.parametrize("fails", ["g++", "hipcc", None])
def test_both_files_are_compiled_before_either_is_replaced(tree, monkeypatch, fails):
    monkeypatch.setattr(hip_build, "torch_ext_missing", lambda: None)
    monkeypatch.setattr(hip_build, "_torch_ext_command", lambda out: ["-o", out])

    def compile_(cmd, what, verbose):
        if what == fails:
            raise RuntimeError(what)
        with open(cmd[cmd.index("-o") + 1], "w") as f:
            f.write("new")

    monkeypatch.setattr(hip_build, "_compile", compile_)
    before = (tree / "_bl_torch.x.so").read_bytes()
    if fails:
        with pytest.raises(RuntimeError):
            hip_build.build()
        assert (tree / "lib.so").read_text() == "old" and (tree / "_bl_torch.x.so").read_bytes() == before
    else:
        hip_build.build()
        assert (tree / "lib.so").read_text() == (tree / "_bl_torch.x.so").read_text() == "new"


def test_the_library_is_built_without_the_tools_of_the_extension(tree, monkeypatch):
    monkeypatch.setattr(hip_build, "torch_ext_missing", lambda: "no g++")
    monkeypatch.setattr(hip_build, "_compile", lambda cmd, what, verbose: open(cmd[cmd.index("-o") + 1], "w").close())
    with pytest.warns(RuntimeWarning, match="no g"):
        hip_build.build()
    assert (tree / "lib.so").read_text() == "" and not (tree / "_bl_torch.x.so").exists()


def test_other_build_flags_make_the_build_stale(tree, monkeypatch):
    """The flags stand in build.py itself."""
    (tree / "build.py").write_text("")
    os.utime(str(tree / "build.py"), (1000, 1000))
    monkeypatch.setattr(hip_build, "__file__", str(tree / "build.py"))
    monkeypatch.setattr(hip_build, "torch_ext_missing", lambda: None)
    assert not hip_build.is_stale()
    os.utime(str(tree / "build.py"), (1e10, 1e10))
    assert hip_build.is_stale()
    os.utime(str(tree / "_bl_torch.x.so"), (2e10, 2e10))
    assert hip_build.is_stale()                                      # the library
    os.utime(str(tree / "lib.so"), (2e10, 2e10))
    assert not hip_build.is_stale()
    os.utime(str(tree / "_bl_torch.x.so"), (1000, 1000))
    assert hip_build.is_stale()                                      # the extension
