"""The stream that the binding takes when none is named."""
import pytest
import torch

from paper_2210_08804_amd import binding as B


def test_a_forked_child_is_refused(monkeypatch):
    """A child forked from a process that uses the GPU cannot: torch says so, and the binding asks it at every call, also
    behind calls that went well."""
    monkeypatch.setattr(torch.cuda, "_initialized", True)
    monkeypatch.setattr(B, "_device", lambda: 0)
    monkeypatch.setattr(B, "_raw_stream", lambda device: 1234)
    assert B._stream(None) == 1234
    monkeypatch.setattr(torch.cuda, "_is_in_bad_fork", lambda: True)
    with pytest.raises(RuntimeError, match="fork"):
        B._stream(None)
