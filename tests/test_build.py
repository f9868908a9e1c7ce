"""The C library is built and usable without its Python front end's native marshalling: neither a failure of that extension nor a
missing torch keeps libpe.so from being built, and the front end works through ctypes without it."""
import os
import subprocess
import sys

import pytest
import torch

import paper_2509_04377_amd as package
from paper_2509_04377_amd import binding as pe
from paper_2509_04377_amd import build


@pytest.fixture
def small(tmp_path, monkeypatch):
    """The build of a library of one function, under tmp_path."""
    (tmp_path / "one.hip").write_text('extern "C" int one() { return 1; }\n')
    monkeypatch.setattr(build, "CSRC", str(tmp_path))
    monkeypatch.setattr(build, "BUILD", str(tmp_path / "o"))
    monkeypatch.setattr(build, "SOURCES", ["one.hip"])
    monkeypatch.setattr(build, "LIB", str(tmp_path / "lib.so"))
    monkeypatch.setattr(build, "HOST_LIB", str(tmp_path / "host.so"))
    monkeypatch.setattr(build, "build_c_smoke", lambda: None)
    return tmp_path


def test_library_is_built_where_the_extension_fails(small):
    (small / "pe_host.cpp").write_text("this is no C++\n")
    with pytest.raises(RuntimeError, match="g\\+\\+ failed on pe_host.cpp"):
        build.build()
    assert os.path.exists(build.LIB) and not os.path.exists(build.HOST_LIB)


def test_library_is_built_without_torch(small, monkeypatch):
    monkeypatch.setitem(sys.modules, "torch", None)
    assert build.build() == build.LIB
    assert os.path.exists(build.LIB) and not os.path.exists(build.HOST_LIB)


def test_build_script_imports_no_torch():
    code = "import sys; sys.modules['torch'] = None; sys.path.insert(0, %r); import build" % os.path.dirname(build.__file__)
    subprocess.run([sys.executable, "-c", code], check=True)


def _host_of_a_fresh_load(monkeypatch):
    monkeypatch.setattr(pe, "_lib", None)
    monkeypatch.setattr(pe, "_host", None)
    with pytest.warns(RuntimeWarning, match="_pe_host.so"):
        assert pe.pe_version() >= 100
    return pe._host


def test_front_end_without_the_extension(monkeypatch, tmp_path):
    monkeypatch.setattr(pe, "HOST_PATH", str(tmp_path / "none.so"))
    assert _host_of_a_fresh_load(monkeypatch).paged_decode(1, 2, 3) is None
    desc = pe.make_desc(torch.float32, 1, 1, 1, 64, 16, 1, 1)
    t = torch.zeros(1)
    with pytest.raises(ValueError, match="q must be a GPU tensor"):
        pe.pe_paged_decode(desc, t, t, t, t, t, 1.0, t)


def test_front_end_with_an_extension_that_does_not_load(monkeypatch):
    pe.lib()
    monkeypatch.delattr(package, "_pe_host", raising=False)
    monkeypatch.setitem(sys.modules, package.__name__ + "._pe_host", None)
    assert isinstance(_host_of_a_fresh_load(monkeypatch), pe._NoHost)
