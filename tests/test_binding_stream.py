"""The stream a call is enqueued on: torch's current one, found again by every call; in a forked child, where torch refuses to
use the GPU, the refusal reaches the caller.  Stand-ins for torch's functions: no GPU needed."""
import os
from types import SimpleNamespace

import pytest

torch = pytest.importorskip("torch")

from paper_2508_08256_amd import binding as B  # noqa: E402


@pytest.fixture
def handles(monkeypatch):
    parent, now = os.getpid(), {"device": 0, 0: 7, 1: 9}

    def current_stream():
        if os.getpid() != parent:
            raise RuntimeError("cannot use the GPU in a forked process")
        return SimpleNamespace(cuda_stream=now[now["device"]])

    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: now["device"], raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: now[d], raising=False)
    monkeypatch.setattr(B, "_current_stream", None)
    return now


def test_every_call_asks_for_the_current_stream(handles):
    assert B._stream() == 7
    handles[0] = 11
    assert B._stream() == 11
    handles["device"] = 1
    assert B._stream() == 9


def test_a_forked_child_is_refused(handles):
    assert B._stream() == 7
    pid = os.fork()
    if pid == 0:
        try:
            B._stream()
        except RuntimeError:
            os._exit(3)
        os._exit(0)
    assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 3
    assert B._stream() == 7
