"""A process that was forked from one that uses the GPU cannot use it: a call there is refused by torch, as
torch.cuda.current_stream() is, before the library sees it.  Without a GPU: what torch knows of the fork is set by hand."""
import pytest
import torch

from paper_2505_23317_amd.cfdetr import Encoder


def _as_if(monkeypatch, forked):
    monkeypatch.setattr(torch.cuda, "_initialized", True)
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: forked)
    for name, value in (("_cuda_isInBadFork", lambda: forked), ("_cuda_getDevice", lambda: 0),
                        ("_cuda_getCurrentRawStream", lambda device: 1234 + device)):
        monkeypatch.setattr(torch._C, name, value, raising=False)


def test_refused_in_a_forked_child(monkeypatch):
    _as_if(monkeypatch, forked=True)
    with pytest.raises(RuntimeError, match="forked subprocess"):
        torch.cuda.current_stream()
    with pytest.raises(RuntimeError, match="forked subprocess"):
        Encoder._stream()


def test_the_number_elsewhere(monkeypatch):
    _as_if(monkeypatch, forked=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: pytest.fail("an object was made"))
    assert Encoder._stream() == 1234
