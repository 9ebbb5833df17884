"""GPU parity of the neighbour searches on points that are not finite or whose
distances over- or underflow: the grid against the brute-force kernel bit for
bit, and the neighbours of a cloud's own points, by thread and by wave, against
keys (d2, index) sorted by torch.  (A NaN distance has the sign that its
operands give it, so which of several NaN distances comes first is not held;
the points are.)"""
import numpy as np
import pytest

import workloads
from _grid_clouds import clouds
from _odd_clouds import odd_cloud

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


@pytest.mark.parametrize("odd", ["queries", "points", "both"])
@pytest.mark.parametrize("name,K", [("nan", 1), ("nan coordinate", 4), ("inf", 4), ("far", 8), ("huge", 1), ("tiny", 9),
                                    ("nan axis", 4), ("inf axis", 1), ("all nan", 4)])
def test_topk_by_grid_and_by_brute_force(dpr, name, K, odd):
    import torch
    from paper_2205_14330_amd import _abi, chamfer as cf
    a = _t(clouds("ball", 9)[0][:3000] if odd == "queries" else odd_cloud(name, 3000))
    b = _t(clouds("ball", 9)[1][:1100] if odd == "points" else odd_cloud(name, 1100, 1))
    sh = _t(workloads.point_attributes(len(a), 1, K)[0])
    out, idx = cf.topk_sh(a, sh, b, K, with_index=True)
    ref, ridx = torch.empty_like(out), torch.empty_like(idx)
    _abi.check(_abi.load().dpr_topk_sh(len(a), a.data_ptr(), sh.data_ptr(), len(b), b.data_ptr(), 1, K, ref.data_ptr(),
                                       ridx.data_ptr(), torch.cuda.current_stream().cuda_stream))
    assert int(idx.min()) >= 0
    assert torch.equal(idx, ridx) and torch.equal(out, ref)


@pytest.mark.parametrize("odd", ["s1", "s2", "both"])
@pytest.mark.parametrize("name", ["nan", "nan coordinate", "inf", "far", "huge", "tiny", "nan axis", "inf axis",
                                  "all nan"])
def test_chamfer_by_grid_and_by_brute_force(dpr, name, odd):
    """Indices and Eq. (9) as by brute force (with its smaller workspace); the gradient to the order of its FP64 sums."""
    import torch
    from paper_2205_14330_amd import _abi, chamfer as cf
    s1 = _t(clouds("ball", 25)[0][:9000] if odd == "s2" else odd_cloud(name, 9000))
    s2 = _t(clouds("ball", 25)[1][:8900] if odd == "s1" else odd_cloud(name, 8900, 1))
    out = cf.chamfer(s1, s2, grad=True, nn=True)
    L = _abi.load()
    ws = torch.empty(L.dpr_chamfer_ws_bytes(len(s1), len(s2)) // 2, dtype=torch.uint8, device="cuda")
    ref = {k: torch.empty_like(v) for k, v in out.items()}
    _abi.check(L.dpr_chamfer(len(s1), s1.data_ptr(), len(s2), s2.data_ptr(), ref["cd"].data_ptr(), ref["grad2"].data_ptr(),
                             ref["nn12"].data_ptr(), ref["nn21"].data_ptr(), ws.data_ptr(), ws.numel(),
                             torch.cuda.current_stream().cuda_stream))
    assert torch.equal(out["nn12"], ref["nn12"]) and torch.equal(out["nn21"], ref["nn21"])
    assert torch.equal(out["cd"].nan_to_num(-1.0), ref["cd"].nan_to_num(-1.0))
    torch.testing.assert_close(out["grad2"], ref["grad2"], rtol=1e-6, atol=0.0, equal_nan=True)


@pytest.mark.parametrize("K", [4, 9])
@pytest.mark.parametrize("name", ["nan", "nan coordinate", "inf", "far", "huge", "tiny"])
def test_knn_by_thread_and_by_wave(dpr, name, K):
    import torch
    from paper_2205_14330_amd import hybrid
    x = _t(odd_cloud(name, 66000))
    idx, d2 = hybrid.knn(x, K)
    for i in range(0, len(x), 2048):
        d = x[None] - x[i:i + 2048, None]
        d = d * d
        d = (d[..., 0] + d[..., 1]) + d[..., 2]
        r = torch.arange(len(d), device=x.device)
        bits = torch.where(torch.isnan(d), 0x7FC00000, d.view(torch.int32).to(torch.int64))
        key = (bits << 32) | torch.arange(len(x), device=x.device)
        key[r, r + i] = 2 ** 63 - 1
        want = key.topk(K, 1, largest=False).values.sort(1).values & 0xFFFFFFFF
        got = idx[i:i + 2048].long()
        assert int(got.min()) >= 0 and not bool((got == r[:, None] + i).any())
        assert bool((got.sort(1).values.diff(dim=1) > 0).all())
        dg = d.gather(1, got)
        assert torch.equal(dg.nan_to_num(-1.0), d2[i:i + 2048].nan_to_num(-1.0))
        nan = torch.isnan(dg)
        assert torch.equal(nan, torch.isnan(d.gather(1, want)))
        assert torch.equal(got.masked_fill(nan, -1), want.masked_fill(nan, -1)), i
