"""The binding's loading, on the CPU: no call here gets as far as a launch."""
import sys
import threading

import pytest

torch = pytest.importorskip("torch")

import paper_2311_05161_amd as w  # noqa: E402
from paper_2311_05161_amd import binding  # noqa: E402


@pytest.fixture
def unloaded(monkeypatch):
    """The binding as a fresh process has it."""
    monkeypatch.setattr(binding, "_lib", None)
    monkeypatch.setattr(binding, "_native", None)
    monkeypatch.setattr(binding, "_addr", {})


def _refused_call():
    """A call that the binding itself refuses once the library is loaded (a one-dimensional X)."""
    t = torch.zeros(4)
    with pytest.raises(ValueError):
        binding.w4a8_linear(t, None, t, t, t, 64, 128)


def test_first_use_while_another_thread_is_loading(unloaded, monkeypatch):
    cast, inside, go_on, errors = binding.ctypes.cast, threading.Event(), threading.Event(), []

    def slow_cast(*a):
        if threading.current_thread() is loader and not inside.is_set() and slow_cast.left == 0:
            inside.set()
            go_on.wait(60)
        if threading.current_thread() is loader:
            slow_cast.left -= 1
        return cast(*a)

    def load():
        try:
            binding.load_library()
        except Exception as e:   # noqa: BLE001
            errors.append(e)

    slow_cast.left = 2           # the loader stops behind two of the entry points
    loader = threading.Thread(target=load)
    monkeypatch.setattr(binding.ctypes, "cast", slow_cast)
    loader.start()
    assert inside.wait(60)
    try:
        _refused_call()
    finally:
        go_on.set()
        loader.join()
    assert not errors
    _refused_call()


def test_library_loads_without_the_native_marshalling(unloaded, monkeypatch):
    monkeypatch.setitem(sys.modules, w.__name__ + "._native", None)   # import raises ImportError
    monkeypatch.delattr(w, "_native", raising=False)
    with pytest.warns(RuntimeWarning, match="marshalled in Python"):
        lib = binding.load_library()
    assert lib.w4a8_gemm_workspace_bytes(200, 4096, 4096, 128, binding.LAYOUT_TILED) > 0
    assert binding.status_string(binding.ERR_SHAPE)
    _refused_call()
