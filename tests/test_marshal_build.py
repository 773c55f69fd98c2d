"""What the build and the binding do where the extension module cannot be built: the libraries are there all the same, and
the binding does its marshalling in Python."""
import os
import sys

from paper_2512_18134_amd import binding, build


def test_the_module_is_left_out_without_torch(tmp_path, monkeypatch):
    path = str(tmp_path / "_marshal.so")
    open(path, "w").close()                          # an older one is not left behind
    monkeypatch.setattr(build, "MARSHAL_PATH", path)
    monkeypatch.setitem(sys.modules, "torch", None)  # importing it raises ImportError
    assert build._compile_marshal(False) is None and not os.path.exists(path)


def test_the_libraries_come_before_the_module(monkeypatch):
    done = []

    def fail(verbose):
        raise RuntimeError("no module")

    monkeypatch.setattr(build, "generate_sources", lambda verbose: None)
    monkeypatch.setattr(build, "_compile", lambda path, extra, verbose: done.append(path))
    monkeypatch.setattr(build, "_compile_marshal", fail)
    try:
        build.build_library()
    except RuntimeError:
        pass
    assert done == [build.LIB_PATH, build.DEBUG_LIB_PATH]


def test_the_module_needs_no_other_compiler(monkeypatch):
    seen = []
    monkeypatch.setenv("CXX", "/no/such/compiler")
    monkeypatch.setattr(build, "MARSHAL_PATH", "/no/such/path")
    monkeypatch.setattr(build, "_run_compiler", lambda cmd, *rest: seen.append(cmd[0]))
    build._compile_marshal(False)
    assert seen == [build._hipcc()]


def test_without_the_module_every_call_is_handed_back(monkeypatch):
    monkeypatch.setattr(binding, "MARSHAL_PATH", "/no/such/path")
    monkeypatch.setattr(binding, "_marshal_module", None)
    native = binding._native()
    assert native.fwd(0) is None and native.splitkv(0) is None and native.bwd(0) is None
    monkeypatch.undo()
    assert binding._native() is not native
