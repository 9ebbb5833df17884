"""dpr_knn, dpr_hybrid_update and dpr_chamfer with a workspace of exactly the
size they report that begins 8 bytes past a 16-byte boundary, with a marker
behind it."""
import ctypes

import numpy as np
import pytest

import workloads
from _grid_clouds import clouds

pytestmark = pytest.mark.gpu


def _ws(nbytes):
    import torch
    buf = torch.full((nbytes + 64,), 0x5A, dtype=torch.uint8, device="cuda")
    assert buf.data_ptr() % 16 == 0
    return buf, buf.data_ptr() + 8, lambda: bool((buf[nbytes + 8:] == 0x5A).all() and (buf[:8] == 0x5A).all())


def test_workspaces_off_16_bytes():
    import torch
    import paper_2205_14330_amd as dpr
    from paper_2205_14330_amd import _abi, chamfer as cf, hybrid
    L, st = _abi.load(), torch.cuda.current_stream().cuda_stream
    s1, s2 = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in clouds("surface", 25))
    n1, n2, K = len(s1), len(s2), 8
    idx, d2 = hybrid.knn(s1, K)
    nb = L.dpr_knn_ws_bytes(n1, K)
    buf, ws, whole = _ws(nb)
    i, d = torch.empty_like(idx), torch.empty_like(d2)
    _abi.check(L.dpr_knn(n1, s1.data_ptr(), K, i.data_ptr(), d.data_ptr(), ws, nb, st))
    assert torch.equal(i, idx) and torch.equal(d, d2) and whole()

    want = cf.chamfer(s1, s2, nn=True)
    nb = L.dpr_chamfer_ws_bytes(n1, n2)
    buf, ws, whole = _ws(nb)
    out = {k: torch.empty_like(v) for k, v in want.items()}
    _abi.check(L.dpr_chamfer(n1, s1.data_ptr(), n2, s2.data_ptr(), *(out[k].data_ptr() for k in ("cd", "grad2", "nn12", "nn21")),
                             ws, nb, st))
    assert all(torch.equal(out[k], want[k]) for k in ("cd", "nn12", "nn21")) and whole()

    sc = dpr.SceneTensors(s1, *(torch.from_numpy(a).float().cuda() for a in workloads.point_attributes(n1, 1, 2)))
    ref, counts = hybrid.hybrid_update(sc, 48, K, 0.02)
    nb = L.dpr_hybrid_ws_bytes(n1, 1, K)
    buf, ws, whole = _ws(nb)
    o = dpr.SceneTensors(*(torch.empty((2 * n1,) + tuple(t.shape[1:]), device="cuda") for t in (sc.xyz, sc.sh, sc.opacity, sc.radius)))
    c = (ctypes.c_int64 * 3)()
    _abi.check(L.dpr_hybrid_update(n1, 1, sc.xyz.data_ptr(), sc.sh.data_ptr(), sc.opacity.data_ptr(), sc.radius.data_ptr(), 48, K,
                                   0.02, o.xyz.data_ptr(), o.sh.data_ptr(), o.opacity.data_ptr(), o.radius.data_ptr(), c, ws, nb, st))
    assert list(c) == [counts["voxels"], counts["kept"], counts["points"]] and whole()
    for a in ("xyz", "sh", "opacity", "radius"):
        assert torch.equal(getattr(o, a)[:c[2]], getattr(ref, a))
