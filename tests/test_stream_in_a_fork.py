"""A process that was forked after its parent had initialised the GPU cannot use it: a call there is refused by torch, as
torch.cuda.current_stream() is, before the library sees it.  Without a GPU: what torch knows of the fork is set by hand."""
import pytest
import torch

from paper_2505_23317_amd.cfdetr import Encoder


def _as_if(monkeypatch, initialised, forked):
    monkeypatch.setattr(torch.cuda, "_initialized", initialised)
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: forked)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 0, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 1234 + device, raising=False)


def test_refused_in_a_forked_child(monkeypatch):
    _as_if(monkeypatch, initialised=True, forked=True)
    with pytest.raises(RuntimeError, match="forked subprocess"):
        torch.cuda.current_stream()
    with pytest.raises(RuntimeError, match="forked subprocess"):
        Encoder._stream()


def test_initialises_first(monkeypatch):
    """A process that has not used the GPU yet goes the ordinary way, which initialises it."""
    _as_if(monkeypatch, initialised=False, forked=False)
    asked = []

    class Stream:
        cuda_stream = 77

    monkeypatch.setattr(torch.cuda, "current_stream", lambda: asked.append(1) or Stream())
    assert Encoder._stream() == 77 and asked == [1]


def test_the_number_where_the_gpu_is_in_use(monkeypatch):
    _as_if(monkeypatch, initialised=True, forked=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: pytest.fail("an object was made"))
    assert Encoder._stream() == 1234
