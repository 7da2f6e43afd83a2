"""Loading the native marshaller: only one made for this interpreter and torch is used, and none that fails to load stops a call.
Building: the C-ABI library stands without it."""
import os
import warnings

import pytest

torch = pytest.importorskip("torch")

from paper_2603_08713_amd import binding, build  # noqa: E402


@pytest.fixture
def made():
    if not os.path.exists(build.MARSHAL_LIB):
        pytest.skip("no native marshaller here")


def test_made_for_this_torch(made):
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        assert binding._load_native(torch) is not None


def test_made_for_another(made, monkeypatch):
    monkeypatch.setattr(binding, "marshal_tag", lambda t: "cpython-399-none torch-0")
    with pytest.warns(UserWarning, match="built for .*ctypes"):
        assert binding._load_native(torch) is None


@pytest.mark.parametrize("content", [None, b"", b"not a library"])
def test_missing_or_broken(monkeypatch, tmp_path, content):
    path = tmp_path / "_marshal.so"
    monkeypatch.setattr(binding, "_MARSHAL_PATH", str(path))
    if content is None:
        assert binding._load_native(torch) is None
        return
    path.write_bytes(content)
    with pytest.warns(UserWarning, match="ctypes"):
        assert binding._load_native(torch) is None


def test_build_without_the_host_compiler(monkeypatch, tmp_path, capsys):
    stale = tmp_path / "_marshal.so"
    stale.write_bytes(b"older")
    monkeypatch.setattr(build, "MARSHAL_LIB", str(stale))
    monkeypatch.setattr(build.shutil, "which", lambda name: None if name == "g++" else "/usr/bin/" + os.path.basename(name))
    build.build_marshal()
    assert "not built: no g++" in capsys.readouterr().out and not stale.exists()


def test_build_names_the_tool_that_failed(monkeypatch, tmp_path):
    monkeypatch.setattr(build, "MARSHAL_LIB", str(tmp_path / "_marshal.so"))
    monkeypatch.setattr(build, "MARSHAL_SRC", str(tmp_path / "absent.cpp"))
    with pytest.raises(RuntimeError, match=r"^g\+\+ failed"):
        build.build_marshal()
