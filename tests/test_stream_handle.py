"""The stream a call goes to when the caller names none: torch's current one, whatever way the binding asks for it."""
import os
import threading
import types

import pytest

torch = pytest.importorskip("torch")

from paper_2602_03537_amd import binding  # noqa: E402


@pytest.fixture
def fake_torch(monkeypatch):
    """Stands in for the device side of torch: the current device, its streams, and how often torch was asked to initialise."""
    state = types.SimpleNamespace(device=0, handles={0: 0x1000, 1: 0x2000}, asked=0, bad_fork=False)

    def current_stream():
        state.asked += 1
        if state.bad_fork:
            raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")
        return types.SimpleNamespace(cuda_stream=state.handles[state.device])
    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: state.device, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: state.handles[d], raising=False)
    monkeypatch.setattr(binding, "_raw_stream", None)
    return state


@pytest.mark.parametrize("private_names", [True, False])
def test_handle_follows_the_current_device_and_stream(fake_torch, monkeypatch, private_names):
    if not private_names:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert binding._stream() == 0x1000
    fake_torch.handles[0] = 0x1100           # another stream became current
    assert binding._stream() == 0x1100
    fake_torch.device = 1                    # another device
    assert binding._stream() == 0x2000
    assert binding._stream(types.SimpleNamespace(cuda_stream=0x77)) == 0x77
    if private_names:
        assert fake_torch.asked == 1         # torch initialises the device once


@pytest.mark.parametrize("private_names", [True, False])
def test_forked_child_is_refused_by_torch(fake_torch, monkeypatch, private_names):
    # torch refuses the GPU in a child forked after its initialisation; a handle remembered from the parent would go round that
    if not private_names:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream")
    assert binding._stream() == 0x1000
    pid = os.fork()
    if pid == 0:
        code = 1
        try:
            fake_torch.bad_fork = True
            for _ in range(2):
                try:
                    binding._stream()
                    os._exit(2)
                except RuntimeError:
                    pass
            code = 0
        finally:
            os._exit(code)
    _, status = os.waitpid(pid, 0)
    assert os.waitstatus_to_exitcode(status) == 0
    assert binding._stream() == 0x1000       # the parent goes on


@pytest.mark.gpu
def test_handle_is_torchs_on_every_stream_and_thread():
    binding._stream()
    side = torch.cuda.Stream()
    got = {}

    def ask(name, stream):
        with torch.cuda.stream(stream):
            got[name] = binding._stream()
    for name, stream in (("default", torch.cuda.default_stream()), ("side", side)):
        t = threading.Thread(target=ask, args=(name, stream))
        t.start()
        t.join()
        ask(name + " here", stream)
    assert got == {"default": torch.cuda.default_stream().cuda_stream, "default here": torch.cuda.default_stream().cuda_stream,
                   "side": side.cuda_stream, "side here": side.cuda_stream}
    assert binding._stream(side) == side.cuda_stream
