"""The autograd form gives its device memory back: a render whose outputs are
dropped, with or without a backward, leaves nothing allocated."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("backward", [False, True])
@pytest.mark.parametrize("mode", ["stored", "recompute"])
def test_render_frees_its_buffers(backward, mode):
    import gc
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_14330_amd as dpr
    sc = dpr.SceneTensors.from_numpy(workloads.small_scene(3, 3000, extent=0.6))
    cams = [workloads.random_sphere_camera(np.random.default_rng(1), 70, 50) for _ in range(2)]
    xyz = sc.xyz.clone().requires_grad_(True)

    def step():
        img, tr = dpr.render(xyz, sc.sh, sc.opacity, sc.radius, cams, dpr.RenderParams(bwd_mode=mode))
        if backward:
            torch.autograd.grad(img.sum() + tr.sum(), xyz)

    step()
    gc.collect()
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    for _ in range(3):
        step()
    gc.collect()
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == before
