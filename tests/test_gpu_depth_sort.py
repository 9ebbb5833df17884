"""The depth sort at the edges of its blocks, digits and paths: the plan's
sorted keys and item order against a stable numpy sort of the float32 depths,
exactly."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dpr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_14330_amd as d
    d.load()
    return d


def _depths(kind, n, rng):
    if kind == "near":                      # within an octave or two: narrow digits
        z = rng.uniform(1.3, 4.7, n)
    elif kind == "wide":                    # most of the float range: 11-bit digits
        z = np.exp(rng.uniform(np.log(0.011), np.log(1e12), n))
    elif kind == "ties":                    # few distinct depths, and some behind the camera
        z = rng.integers(-1, 3, n).astype(np.float64)
    elif kind == "same":
        z = np.full(n, 2.0)
    else:                                   # every item dropped
        z = np.full(n, -1.0)
    return z.astype(np.float32)


def _plan_order(dpr, scenes, views):
    import torch
    plan = dpr.Plan(scenes, views, dpr.RenderParams())
    inf = plan.info()
    take = lambda off: plan.plan_ws[off:off + 4 * inf.items].view(torch.int32).cpu().numpy().view(np.uint32)
    out = take(inf.key_off).copy(), take(inf.order_off).copy()
    plan.forward()
    torch.cuda.synchronize()
    return out


def _expected(z, item_off):
    key = np.where(z > np.float32(0.01), z.view(np.uint32), np.uint32(0xFFFFFFFF))
    order = np.argsort(key, kind="stable")
    return key[order], (order + item_off).astype(np.uint32)


def _scene(dpr, z, rng):
    n = len(z)
    xyz = np.zeros((n, 3), np.float32)      # on the axis: in view at any depth
    xyz[:, 2] = z
    return dpr.SceneTensors.from_numpy(workloads.Scene(xyz, np.zeros((n, 1, 3), np.float32), np.full(n, 0.5, np.float32),
                                                       np.full(n, 0.02, np.float32)))


def _camera(size=40):
    c = workloads.Camera(np.eye(3), np.zeros(3), 50.0, 50.0, size / 2 + 0.5, size / 2 + 0.5, size, size)
    return c


@pytest.mark.parametrize("kind", ["near", "wide", "ties", "same", "dropped"])
@pytest.mark.parametrize("n", [1, 64, 129, 8192, 8193, 16384, 41000])
def test_order(dpr, kind, n):
    rng = np.random.default_rng(n)
    z = _depths(kind, n, rng)
    keys, order = _plan_order(dpr, [_scene(dpr, z, rng)], [(0, _camera())])
    rk, ro = _expected(z, 0)
    assert np.array_equal(keys, rk) and np.array_equal(order, ro)


def test_views_of_different_sizes_and_ranges(dpr):
    """One plan with views of less than a block, of several blocks, of no item, and of digits of different width."""
    rng = np.random.default_rng(5)
    zs = [_depths("near", 20000, rng), _depths("wide", 3000, rng), np.zeros(0, np.float32), _depths("ties", 8193, rng),
          _depths("wide", 30011, rng)]
    scenes = [_scene(dpr, z, rng) for z in zs]
    views = [(i, _camera(24 + i)) for i in (0, 4, 1, 2, 3, 0)]
    keys, order = _plan_order(dpr, scenes, views)
    off = 0
    for i, _ in views:
        rk, ro = _expected(zs[i], off)
        assert np.array_equal(keys[off:off + len(rk)], rk) and np.array_equal(order[off:off + len(ro)], ro)
        off += len(rk)
