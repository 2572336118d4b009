"""A forked child of a process that has used the device is refused by torch; the binding's short way to the current
stream must not get round that.  No GPU: torch's answers are stood in for."""
import os
import types

import torch

from paper_2605_26092_amd import binding


def test_a_forked_child_asks_torch_again(monkeypatch):
    monkeypatch.setattr(binding, "_current_stream", binding._current_stream)          # (put back afterwards)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=5))
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 70 + device)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 1)
    assert [binding._stream(None) for _ in range(3)] == [5, 71, 71]

    def refuse():
        raise RuntimeError("Cannot re-initialize CUDA in forked subprocess")
    monkeypatch.setattr(torch.cuda, "current_stream", refuse)
    child = os.fork()
    if child == 0:
        try:
            binding._stream(None)
        except RuntimeError:
            os._exit(0)
        os._exit(1)
    assert os.waitpid(child, 0)[1] == 0
    assert binding._stream(None) == 71                                                # the parent goes on as before
