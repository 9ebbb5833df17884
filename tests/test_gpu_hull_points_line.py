"""The consistency predicate of given points at the line between its two forms
(an item per lane below 2^22 points, the compacting one from there on)."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu
LINE = 1 << 22


@pytest.mark.parametrize("n,n_cams", [(LINE - 1, 5), (LINE, 1), (LINE + 2049, 6)])
def test_keep_and_filter(n, n_cams):
    import torch
    import paper_2205_14330_amd as dpr
    from paper_2205_14330_amd import hull
    cams = workloads.disc_views(n_cams, size=61)
    masks = workloads.sphere_masks(cams, 0.7)
    xyz = np.random.default_rng(n).uniform(-1, 1, (n, 3)).astype(np.float32)
    xyz[:3] = [[np.nan, 0, 0], [np.inf, 0, 0], [0, -np.inf, 0]]
    want = oracle.hull_consistent(xyz, cams, masks)
    dev = [torch.from_numpy(np.ascontiguousarray(m, np.uint8)).cuda() for m in masks]
    x = torch.from_numpy(xyz).cuda()
    assert np.array_equal(hull.consistency(x, cams, dev).cpu().numpy().astype(bool), want)
    sh, op, rad = torch.randn((n, 1, 3), device="cuda"), torch.rand(n, device="cuda"), torch.rand(n, device="cuda")
    out = hull.consistency_filter(dpr.SceneTensors(x, sh, op, rad), cams, dev)
    sel = torch.from_numpy(want).cuda()
    assert torch.equal(out.xyz, x[sel]) and torch.equal(out.sh, sh[sel])
    assert torch.equal(out.opacity, op[sel]) and torch.equal(out.radius, rad[sel])
