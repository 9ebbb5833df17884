"""Tile lists of splats from one tile to a dozen across, in views of one tile (its
words over many threads), of one band, of several, of bands of part of a row,
and of more tiles than one counting band."""
import numpy as np
import pytest

import oracle
import workloads

from _gpu_util import compare_images, gpu_plan, oparams, random_pixels, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [(16, 16), (130, 150), (400, 400), (8300, 40), (8300, 300)])
def test_wide_splats(size):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_14330_amd as dpr
    w, h = size
    rng = np.random.default_rng(w + h)
    n, f = 700, 200.0
    z = rng.uniform(1.5, 3.0, n)
    px = np.stack([rng.uniform(-20, w + 20, n), rng.uniform(-20, h + 20, n)], 1)
    xyz = np.concatenate([(px - [w / 2, h / 2]) * z[:, None] / f, z[:, None]], 1).astype(np.float32)
    radius = np.exp(rng.uniform(np.log(0.01), np.log(0.4), n)).astype(np.float32)     # 1 to 50 pixels
    sc = workloads.Scene(xyz, rng.standard_normal((n, 4, 3)).astype(np.float32),
                         rng.uniform(0.02, 0.3, n).astype(np.float32), radius)
    cam = workloads.Camera(np.eye(3), np.zeros(3), f, f, w / 2, h / 2, w, h)
    params = dpr.RenderParams()
    plan = gpu_plan([sc], [(0, cam)], params)
    # the rectangles, 16-bit x0, y0, x1, y1 in tiles: small ones, and (in views that allow it) large ones
    inf = plan.info()
    r = to_np(plan.plan_ws[inf.rect_off:inf.rect_off + 8 * n].view(torch.int32)).view(np.uint32).reshape(n, 2)
    span = np.maximum((r[:, 1] & 0xFFFF).astype(int) - (r[:, 0] & 0xFFFF), (r[:, 1] >> 16).astype(int) - (r[:, 0] >> 16))
    assert (span <= 8).any() and ((span > 8).any() or max(size) < 144)
    pix = random_pixels(7, cam, 3000)
    ref = oracle.render(sc, cam, oparams(params), pixels=pix)
    compare_images(to_np(plan.images[0]), to_np(plan.trans[0]), ref, pixels=pix, label=f"{size}")
