"""Eq. (8) kernel where its groups of four floats meet borders: rows of every
length modulo 4 and shorter than a group, images that end inside a group, and
tensors that begin 4, 8 or 12 bytes past a 16-byte boundary."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (2, 1), (5, 1), (9, 2), (1, 2), (4, 3), (7, 5), (3, 341), (2, 342), (5, 797), (700, 1), (3, 2049)]


@pytest.mark.parametrize("lam", [0.0, 0.3])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_loss_edges(lam, offset):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_14330_amd as dpr
    rng = np.random.default_rng(offset)
    R = [rng.standard_normal((h, w, 3)).astype(np.float32) for h, w in SIZES]
    T = [rng.standard_normal((h, w, 3)).astype(np.float32) for h, w in SIZES]

    def place(x, shift):
        buf = torch.full((x.size + 8,), float("nan"), device="cuda")
        out = buf[shift:shift + x.size].view(x.shape)
        out.copy_(torch.from_numpy(x))
        return buf, out

    r = [place(x, offset) for x in R]
    t = [place(x, (2 * offset) % 4) for x in T]
    g = [place(np.zeros_like(x), (offset + 1) % 4 if offset else 0) for x in R]
    loss, _ = dpr.loss_l2_tv([x[1] for x in r], [x[1] for x in t], lam, grads=[x[1] for x in g])
    loss = loss.cpu().numpy()
    u = 2.0 ** -24
    for v in range(len(SIZES)):
        ref_l, ref_g = oracle.loss_l2_tv(R[v], T[v], lam)
        # 12 terms per thread, the block's 8 levels and each term's own roundings, all of one sign
        assert abs(loss[v] - ref_l) <= 32 * u * ref_l, SIZES[v]
        bound = 8 * u * (2 * np.abs(R[v].astype(np.float64) - T[v]) + 4 * lam)
        assert (np.abs(g[v][1].cpu().numpy() - ref_g) <= bound).all(), SIZES[v]
        pad = torch.ones(g[v][0].numel(), dtype=torch.bool)      # nothing is written around the gradient
        s = g[v][1].storage_offset()
        pad[s:s + R[v].size] = False
        assert torch.isnan(g[v][0].cpu()[pad]).all(), SIZES[v]
