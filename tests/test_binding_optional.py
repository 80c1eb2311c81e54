"""The binding's native module is an option: without it, or with one that does
not load, the library loads and the Python code makes every call."""
import warnings

import pytest


@pytest.fixture
def fresh(monkeypatch):
    import os

    from paper_2112_10034_amd import cox

    if not os.path.exists(cox.LIB_PATH):
        import __graft_entry__

        __graft_entry__.build()
    monkeypatch.setattr(cox, "_lib", None)
    monkeypatch.setattr(cox, "_native", None)
    return cox


@pytest.mark.parametrize("content", [None, b"", b"not a shared library"])
def test_without_the_native_module(fresh, monkeypatch, tmp_path, content):
    path = tmp_path / "_coxbind.so"
    if content is not None:
        path.write_bytes(content)
    monkeypatch.setattr(fresh, "_BIND_PATH", str(path))
    with pytest.warns(UserWarning, match="does not load"):
        L = fresh.lib()
    assert L.cox_version() >= 100
    assert fresh._native.scan(1, 2, 3) is None and fresh._native.segmented() is None
    with pytest.raises(TypeError):
        fresh.warp_scan([1, 2])


def test_the_built_module_loads_without_a_warning(fresh):
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        fresh.lib()
    assert type(fresh._native).__name__ == "module"


def test_a_failing_binding_compiler_leaves_the_library_built(monkeypatch, tmp_path):
    from paper_2112_10034_amd import build_lib

    stale = tmp_path / "_coxbind.so"
    stale.write_bytes(b"stale")
    monkeypatch.setattr(build_lib, "BIND", str(stale))
    monkeypatch.setattr(build_lib, "SOURCES", [])
    monkeypatch.setenv("CXX", "false")
    monkeypatch.setattr(build_lib, "HIPCC", "true")  # links nothing; its output lies ready
    monkeypatch.setattr(build_lib, "LIB", str(tmp_path / "libcox.so"))
    (tmp_path / "libcox.so.tmp").write_bytes(b"library")
    with pytest.warns(UserWarning, match="not built"):
        build_lib.build(jobs=1)
    assert (tmp_path / "libcox.so").exists() and not stale.exists()
