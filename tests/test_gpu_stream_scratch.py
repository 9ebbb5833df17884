"""A call on a stream of its own keeps its scratch to itself: tensors made on the
current stream right after the call returns do not disturb it."""
import pytest

import workloads
from _grid_clouds import clouds

pytestmark = pytest.mark.gpu


def test_calls_on_another_stream():
    import torch
    from paper_2205_14330_amd import chamfer as cf
    from paper_2205_14330_amd import hybrid
    s1, s2 = (torch.from_numpy(a).cuda() for a in clouds("surface", 25))
    sh = torch.from_numpy(workloads.point_attributes(len(s1), 1, 1)[0]).float().cuda()
    calls = [lambda s: cf.topk_sh(s1, sh, s2, 4, with_index=True, stream=s),
             lambda s: tuple(cf.chamfer(s1, s2, grad=False, nn=True, stream=s).values()),
             lambda s: hybrid.knn(s1, 8, stream=s)]
    for call in calls:
        want = call(None)
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        got = call(side)
        junk = [torch.full((1 << k,), 0xA5, dtype=torch.uint8, device="cuda") for k in range(9, 25) for _ in range(3)]
        side.synchronize()
        torch.cuda.synchronize()
        assert all(torch.equal(g, w) for g, w in zip(got, want)) and len(junk) == 48
