"""Scratch memory of a call or a plan on a given stream comes from that stream's pool: it
is dropped when the call returns, while its kernels still run, and memory of
another stream's pool could be handed to that stream's next tensor.  Checked on
the CPU with a stand-in for the library and for the stream context."""
import contextlib

import pytest
import torch

import workloads
from paper_2205_14330_amd import chamfer, hull, hybrid, renderer
from paper_2205_14330_amd.renderer import SceneTensors


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


def _scene():
    return SceneTensors(_dev(9, 3), _dev(9, 4, 3), _dev(9), _dev(9))


def _views():
    return [workloads.orbit_camera(0, 8, 8, 6)], [torch.zeros(6, 8, dtype=torch.uint8).as_subclass(_Cuda)]


CALLS = {
    "topk_sh": _topk,
    "chamfer": lambda s: chamfer.chamfer(_dev(9, 3), _dev(5, 3), stream=s),
    "knn": lambda s: hybrid.knn(_dev(9, 3), 4, stream=s),
    "voxel_reduce": lambda s: hybrid.voxel_reduce(_scene(), 4, stream=s),
    "hybrid_update": lambda s: hybrid.hybrid_update(_scene(), 4, 4, 0.1, stream=s),
    "hull_sample": lambda s: hull.hull_sample(*_views(), (0, 0, 0), (1, 1, 1), 1, 9, stream=s),
    "consistency": lambda s: hull.consistency(_dev(9, 3), *_views(), stream=s),
    "consistency_filter": lambda s: hull.consistency_filter(_scene(), *_views(), stream=s),
    "loss_l2_tv with a Workspace": lambda s: renderer.loss_l2_tv([_dev(6, 8, 3)], [_dev(6, 8, 3)], stream=s,
                                                                 workspace=renderer.Workspace("cpu")),
    "loss_l2_tv": lambda s: renderer.loss_l2_tv([_dev(6, 8, 3)], [_dev(6, 8, 3)], stream=s),
}


def _plan(workspace):
    def call(s):
        cam = workloads.orbit_camera(0, 8, 8, 6)
        p = renderer.Plan([_scene()], [(0, cam)], stream=s, workspace=workspace() if workspace else None)
        p.forward()
        p.backward([_dev(6, 8, 3)])
    return call


PLANS = {"plan": _plan(None), "plan with a Workspace": _plan(lambda: renderer.Workspace("cpu"))}


@pytest.mark.parametrize("name", sorted(CALLS) + sorted(PLANS))
def test_scratch_is_allocated_on_the_calls_stream(monkeypatch, name):
    current, scratch = [None], []
    empty = torch.empty

    @contextlib.contextmanager
    def stream(s):
        current.append(s)
        yield
        current.pop()

    def recorded(*a, **k):
        if k.get("dtype") == torch.uint8 and a in ((1024,), (1 << 21,)):
            scratch.append(current[-1])
        return empty(*a, **k)

    for module in (chamfer, hybrid, hull, renderer):
        monkeypatch.setattr(module, "load", _Lib)
    monkeypatch.setattr(torch.cuda, "stream", stream)
    monkeypatch.setattr(torch, "empty", recorded)
    side = _Stream()
    (CALLS.get(name) or PLANS[name])(side)
    assert scratch == [side] * (3 if name in PLANS else 1)
