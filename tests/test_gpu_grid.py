"""GPU parity of the grid searches at the edges of their rules: the Chamfer
distance and the top-k transfer of the video warm start on clouds above the
sizes from which the grid is searched, and the neighbour search by thread and
by wave.  Indices bit for bit (against the oracle, or against keys
(d2 bits, index) sorted by torch from the same float32 operations); Eq. (9) to
1e-12; the gradient to float32 rounding."""
import ctypes

import numpy as np
import pytest

import oracle
import workloads
from _grid_clouds import NAMES, clouds

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dpr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_14330_amd as d
    d.load()
    return d


def _t(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def _nearest(q, c, K, skip_self=False):
    """The K smallest (d2, index) per query, from float32 distances with each operation rounded."""
    import torch
    out = []
    for i in range(0, q.shape[0], 1024):
        x = q[i:i + 1024, None, :] - c[None]
        x = x * x
        d = (x[..., 0] + x[..., 1]) + x[..., 2]
        key = (d.view(torch.int32).to(torch.int64) << 32) | torch.arange(c.shape[0], device=q.device)
        if skip_self:
            r = torch.arange(d.shape[0], device=q.device)
            key[r, r + i] = 2 ** 63 - 1
        out.append((key.topk(K, 1, largest=False).values & 0xFFFFFFFF).to(torch.int32))
    return torch.cat(out)


@pytest.mark.parametrize("name", NAMES)
def test_chamfer_by_grid(dpr, name):
    from paper_2205_14330_amd import chamfer as cf
    s1, s2 = clouds(name, 25)                    # 10000 points; "one" stays on the brute-force side
    out = cf.chamfer(_t(s1), _t(s2), grad=True, nn=True)
    assert np.array_equal(out["nn12"].cpu().numpy(), oracle.chamfer_nn(s1, s2)[0])
    assert np.array_equal(out["nn21"].cpu().numpy(), oracle.chamfer_nn(s2, s1)[0])
    rcd, rg = oracle.chamfer(s1, s2)
    assert float(out["cd"].cpu()[0]) == pytest.approx(rcd, rel=1e-12, abs=1e-300)
    np.testing.assert_allclose(out["grad2"].cpu().numpy(), rg, rtol=1e-6, atol=1e-7 * max(np.abs(rg).max(), 1e-30))


def test_chamfer_with_the_brute_force_workspace(dpr):
    """A workspace of the brute-force search's size is still accepted at any size, with the same results."""
    import torch
    from paper_2205_14330_amd import _abi, chamfer as cf
    s1, s2 = (_t(a) for a in clouds("surface", 25))
    n1, n2 = len(s1), len(s2)
    up = lambda x: (x + 255) // 256 * 256
    small = (up(8 * n1) + up(8 * n2) + up(24 * n2) + up(4 * n2) + up(8 * ((n1 + 255) // 256)) +
             up(8 * ((n2 + 255) // 256)))
    L = _abi.load()
    assert small < L.dpr_chamfer_ws_bytes(n1, n2)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    cd = torch.empty(1, dtype=torch.float64, device="cuda")
    nn12 = torch.empty(n1, dtype=torch.int32, device="cuda")
    args = (n1, s1.data_ptr(), n2, s2.data_ptr(), cd.data_ptr(), None, nn12.data_ptr(), None, ws.data_ptr())
    _abi.check(L.dpr_chamfer(*args, small, torch.cuda.current_stream().cuda_stream))
    ref = cf.chamfer(s1, s2, grad=False, nn=True)
    assert torch.equal(nn12, ref["nn12"]) and torch.equal(cd, ref["cd"])
    assert L.dpr_chamfer(*args, small - 1, None) == 2


@pytest.mark.parametrize("K", [1, 2, 4, 8, 9, 32])
@pytest.mark.parametrize("name", ["surface", "floaters", "clusters", "apart", "thin"])
def test_topk_by_grid(dpr, name, K):
    import torch
    from paper_2205_14330_amd import chamfer as cf
    s1, s2 = clouds(name, 5)
    s2 = s2[:1100]
    deg = K % 4
    sh1 = workloads.point_attributes(len(s1), deg, K)[0]
    out, idx = cf.topk_sh(_t(s1), _t(sh1), _t(s2), K, with_index=True)
    assert torch.equal(idx, _nearest(_t(s2), _t(s1), K))
    acc = np.zeros((len(s2),) + sh1.shape[1:])
    for k in range(K):
        acc += sh1[idx[:, k].cpu().numpy()].astype(np.float64)
    assert np.array_equal(out.cpu().numpy(), (acc / K).astype(np.float32))
    assert torch.equal(cf.topk_sh(_t(s1), _t(sh1), _t(s2), K), out)        # without the indices


@pytest.mark.parametrize("n,K", [(65535, 4), (65536, 2), (65536, 4), (65537, 5), (66000, 8), (66000, 9), (66000, 1)])
@pytest.mark.parametrize("name", ["ball", "surface", "floaters"])
def test_knn_by_thread_and_by_wave(dpr, name, n, K):
    import torch
    from paper_2205_14330_amd import hybrid
    x = _t(clouds(name, 165)[0][:n])
    idx, d2 = hybrid.knn(x, K)
    assert torch.equal(idx, _nearest(x, x, K, True))
    d = x[idx.long()] - x[:, None]
    d = d * d
    assert torch.equal(d2, (d[..., 0] + d[..., 1]) + d[..., 2])


@pytest.mark.parametrize("share", [0.0, 0.02, 0.06, 0.07, 0.3])
def test_update_with_few_and_many_removed(dpr, share):
    """The neighbours among the points left: renumbered where at most one in 16 was removed, searched for anew beyond."""
    from paper_2205_14330_amd import hybrid
    N, K = 64, 6
    x = clouds("floaters", 6)[0]
    sh, op, rad = workloads.point_attributes(len(x), 1, 3)
    c = oracle.Cloud(x, sh, op, rad)
    red = oracle.hybrid_update(c, N, K, 1e30)[0]
    d = np.sort(np.sqrt(((red.xyz[:, None].astype(np.float64) - red.xyz[None]) ** 2).sum(-1)), 1)[:, 1:K + 1]
    s = np.sort(d.std(1))[::-1]
    k = int(round(share * len(s)))
    eps = float(s[0] * 2) if k == 0 else float(0.5 * (s[k - 1] + s[k]))
    ref_red, ref_keep, ref = oracle.hybrid_update(c, N, K, eps)
    got, counts = hybrid.hybrid_update(dpr.SceneTensors.from_numpy(c), N, K, eps)
    assert counts["voxels"] == ref_red.n and counts["kept"] == ref_red.n - k
    for a in ("xyz", "sh", "opacity", "radius"):
        want = np.asarray(getattr(ref, a)).astype(np.float32)
        assert np.array_equal(getattr(got, a).cpu().numpy(), want.reshape(getattr(got, a).shape)), a
