"""The handle of the current stream where torch's short way to it is absent or not to be taken."""
import os
import subprocess
import sys

import pytest
import torch

from paper_2506_19225_amd import vxl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Stream:
    cuda_stream = 0x5150


@pytest.fixture
def device(monkeypatch):
    """A process whose torch says that it has a device set up, and where both ways to the stream only count."""
    calls = []
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: calls.append("public") or Stream())
    monkeypatch.setattr(vxl, "_current_device", lambda: 3)
    monkeypatch.setattr(vxl, "_raw_stream", lambda dev: calls.append(dev) or 0x77)
    return calls


@pytest.mark.parametrize("name", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_imports_where_torch_lacks_the_short_way(name):
    code = f"""
import torch
if hasattr(torch._C, {name!r}):
    del torch._C.{name}
from paper_2506_19225_amd import vxl
class Stream:
    cuda_stream = 0x5150
torch.cuda.is_initialized = lambda: True
torch.cuda.current_stream = lambda: Stream()
assert vxl._stream(None) == 0x5150
"""
    subprocess.run([sys.executable, "-c", code], cwd=ROOT, check=True, timeout=300)


def test_device_not_set_up_takes_the_public_way(device, monkeypatch):
    """Before the first use of the device, and in a child forked after it, where torch raises an error of its own."""
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: False)
    assert vxl._stream(None) == Stream.cuda_stream and device == ["public"]

    def refuse():
        raise RuntimeError("Cannot re-initialize")
    monkeypatch.setattr(torch.cuda, "current_stream", refuse)
    with pytest.raises(RuntimeError, match="Cannot re-initialize"):
        vxl.Layout(0, [0, 4], [0, 0], [])


def test_device_set_up_takes_the_short_way(device, monkeypatch):
    assert vxl._stream(None) == 0x77 and device == [3]
    monkeypatch.setattr(vxl, "_raw_stream", lambda dev: 0)          # the default stream
    assert vxl._stream(None) is None
    assert vxl._stream(Stream()) == Stream.cuda_stream
