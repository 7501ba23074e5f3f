"""The binding's loading, on the CPU: no call here gets as far as a launch."""
import threading

import pytest

torch = pytest.importorskip("torch")

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
