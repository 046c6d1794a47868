"""The binding's extension module is optional and never stale (CPU only): calls
reach the Python marshalling where it cannot be built or loaded, and a module of
another source, C ABI, Python or torch is built anew."""
import os
import shutil
import warnings

import pytest

import paper_2512_13921_amd as swr
from paper_2512_13921_amd import build

torch = pytest.importorskip("torch")


def _refused_in_python():
    """An ordinary call on host tensors: the Python path raises its own error."""
    x = torch.zeros(1, 16, 1, 16)
    with pytest.raises(ValueError, match="x must be a GPU tensor"):
        swr.swr_forward(x, x[..., 0], x, x, 16)


@pytest.fixture()
def unbound(monkeypatch, tmp_path):
    swr.load()
    monkeypatch.setattr(swr, "_native", None)
    monkeypatch.setattr(build, "BINDING", str(tmp_path / "_binding.so"))
    return tmp_path


def test_no_compiler_leaves_the_python_path(unbound, monkeypatch):
    monkeypatch.setenv("PATH", str(unbound))
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        _refused_in_python()
    assert isinstance(swr._native[1], swr._PythonOnly)
    with warnings.catch_warnings():   # said once
        warnings.simplefilter("error")
        _refused_in_python()


def test_a_module_that_does_not_load_leaves_the_python_path(unbound, monkeypatch):
    monkeypatch.setattr(build, "binding_is_current", lambda: True)
    with open(build.BINDING, "wb") as f:
        f.write(b"not a library")
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        _refused_in_python()


def test_a_stale_module_is_not_used(unbound, monkeypatch):
    built = os.path.join(os.path.dirname(build.__file__), "_binding.so")
    if not os.path.exists(built):
        pytest.skip("not built")
    shutil.copy(built, build.BINDING)
    assert build.binding_is_current()
    key = build.binding_key()
    source = unbound / "swr_binding.cpp"
    shutil.copy(build.BINDING_SOURCE, source)
    with open(source, "a") as f:
        f.write("// edited\n")
    for name, path in (("BINDING_SOURCE", str(source)), ("ABI_HEADER", str(source))):
        with monkeypatch.context() as m:
            m.setattr(build, name, path)
            assert build.binding_key() != key and not build.binding_is_current()
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "0.0")
        assert build.binding_key() != key and not build.binding_is_current()
        calls = []
        m.setattr(build, "build_binding", lambda: calls.append(1) or build.BINDING)
        swr._fast()
        assert calls == [1]


def test_each_process_builds_to_a_name_of_its_own():
    assert str(os.getpid()) not in build.BINDING
    assert build._temporary(build.BINDING) == f"{build.BINDING}.tmp{os.getpid():x}"
    assert build._temporary(build.BINDING) in build.binding_command(build._temporary(build.BINDING))
