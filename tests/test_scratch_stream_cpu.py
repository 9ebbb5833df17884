"""Scratch memory of a call on a given stream comes from that stream's pool: it
is dropped when the call returns, while its kernels still run, and memory of
another stream's pool could be handed to that stream's next tensor.  Checked on
the CPU with a stand-in for the library and for the stream context."""
import contextlib

import pytest
import torch

from paper_2205_14330_amd import chamfer


class _Cuda(torch.Tensor):
    """A CPU tensor that says it is on the device."""
    is_cuda = True


def _dev(*shape):
    return torch.zeros(*shape).as_subclass(_Cuda)


class _Lib:
    """Every size query answers 1024 bytes, every call succeeds."""

    def __getattr__(self, name):
        return lambda *a: 1024 if name.endswith("_bytes") else 0


class _Stream:
    cuda_stream = 7


def _topk(stream):
    chamfer.topk_sh(_dev(9, 3), _dev(9, 4, 3), _dev(5, 3), 4, stream=stream)


CALLS = {"topk_sh": _topk}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_scratch_is_allocated_on_the_calls_stream(monkeypatch, name):
    current, scratch = [None], []
    empty = torch.empty

    @contextlib.contextmanager
    def stream(s):
        current.append(s)
        yield
        current.pop()

    def recorded(*a, **k):
        if k.get("dtype") == torch.uint8 and a == (1024,):
            scratch.append(current[-1])
        return empty(*a, **k)

    monkeypatch.setattr(chamfer, "load", _Lib)
    monkeypatch.setattr(torch.cuda, "stream", stream)
    monkeypatch.setattr(torch, "empty", recorded)
    side = _Stream()
    CALLS[name](side)
    assert scratch == [side]
