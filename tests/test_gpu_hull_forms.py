"""The two forms of the consistency predicate (an item per lane; the compacting
one from 2^20 items on) at the line between them, with camera counts that leave
a remainder in either's groups."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
LINE = 1 << 20
LO, HI = np.array([-1, -1, -1], np.float32), np.array([1, 1, 1], np.float32)


@pytest.fixture(scope="module")
def hull():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2205_14330_amd import hull
    return hull


def _dev(masks):
    import torch
    return [torch.from_numpy(np.ascontiguousarray(m, np.uint8)).cuda() for m in masks]


@pytest.mark.parametrize("n,n_cams,capacity", [(LINE - 1, 5, None), (LINE, 1, None), (LINE, 2, 1000),
                                               (LINE + 2047, 3, None), (LINE + 2049, 8, None), (300, 7, None)])
def test_sample(hull, n, n_cams, capacity):
    cams = workloads.disc_views(n_cams, size=61)
    masks = workloads.sphere_masks(cams, 0.6)
    cap = n if capacity is None else capacity
    xyz, kept = hull.hull_sample(cams, _dev(masks), LO, HI, 77, n, capacity=cap)
    rk, ref = oracle.hull_sample(cams, masks, LO, HI, 77, n, capacity=cap)
    assert kept == rk
    assert np.array_equal(xyz.cpu().numpy()[:min(kept, cap)], ref)


@pytest.mark.parametrize("radius", [0.3, 1.0, 1.35, 9.0])      # few to all stay after two cameras: packed, or not
def test_sample_dense_hulls(hull, radius):
    cams = workloads.disc_views(7, size=61)
    masks = workloads.sphere_masks(cams, radius) if radius < 3 else [np.ones((c.height, c.width), np.uint8) for c in cams]
    n = LINE + 300
    xyz, kept = hull.hull_sample(cams, _dev(masks), 0.7 * LO, 0.7 * HI, 78, n, capacity=n)
    rk, ref = oracle.hull_sample(cams, masks, 0.7 * LO, 0.7 * HI, 78, n, capacity=n)
    assert kept == rk
    assert np.array_equal(xyz.cpu().numpy()[:kept], ref)


@pytest.mark.parametrize("n", [255, 257, LINE - 1, LINE + 1])
@pytest.mark.parametrize("degree", [0, 3])
def test_keep_and_filter(hull, n, degree):
    import torch
    import paper_2205_14330_amd as dpr
    cams = workloads.disc_views(3, size=61)
    masks = workloads.sphere_masks(cams, 0.7)
    rng = np.random.default_rng(n)
    xyz = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    xyz[:3] = [[np.nan, 0, 0], [np.inf, 0, 0], [0, -np.inf, 0]]
    want = oracle.hull_consistent(xyz, cams, masks)
    dev = _dev(masks)
    x = torch.from_numpy(xyz).cuda()
    assert np.array_equal(hull.consistency(x, cams, dev).cpu().numpy().astype(bool), want)
    k = (degree + 1) ** 2
    sh = torch.randn((n, k, 3), device="cuda")
    op, rad = torch.rand(n, device="cuda"), torch.rand(n, device="cuda") + 0.1
    out = hull.consistency_filter(dpr.SceneTensors(x, sh, op, rad), cams, dev)
    sel = torch.from_numpy(want).cuda()
    assert torch.equal(out.xyz, x[sel]) and torch.equal(out.sh, sh[sel])
    assert torch.equal(out.opacity, op[sel]) and torch.equal(out.radius, rad[sel])


def test_workspace_grows_with_the_items(hull):
    """A workspace for n items serves fewer, on either side of the line."""
    from paper_2205_14330_amd import _abi
    from paper_2205_14330_amd._abi import load
    from paper_2205_14330_amd.renderer import camera_struct
    c = (_abi.Camera * 1)(camera_struct(workloads.disc_views(1, size=61)[0]))
    sizes = [load().dpr_hull_ws_bytes(n, 1, c) for n in (1, 255, 256, 257, 2048, LINE - 1, LINE, LINE + 1, 1 << 24)]
    assert sizes == sorted(sizes)
