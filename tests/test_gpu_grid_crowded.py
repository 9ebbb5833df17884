"""GPU parity of the k-nearest search where queries are left over by its first
pass (clouds that crowd into a few cells): few of them, a wave each; many, all
queries by brute force; at the sizes from which the grid is searched; and with
points in cell order.  Bit for bit the brute-force kernel's results."""
import numpy as np
import pytest

import workloads
from _grid_clouds import clouds

pytestmark = pytest.mark.gpu


def _check(s1, s2, K):
    import torch
    from paper_2205_14330_amd import _abi, chamfer as cf
    a, b = (torch.from_numpy(np.ascontiguousarray(x, np.float32)).cuda() for x in (s1, s2))
    sh = torch.from_numpy(workloads.point_attributes(len(a), 1, K)[0]).float().cuda()
    out, idx = cf.topk_sh(a, sh, b, K, with_index=True)
    ref, ridx = torch.empty_like(out), torch.empty_like(idx)
    _abi.check(_abi.load().dpr_topk_sh(len(a), a.data_ptr(), sh.data_ptr(), len(b), b.data_ptr(), 1, K, ref.data_ptr(),
                                       ridx.data_ptr(), torch.cuda.current_stream().cuda_stream))
    assert torch.equal(idx, ridx) and torch.equal(out, ref)


@pytest.mark.parametrize("K", [1, 3, 8, 9])
@pytest.mark.parametrize("n2,share", [(1100, 0.2), (1100, 1.0), (8191, 1.0), (8192, 0.0), (8192, 0.49), (8192, 0.51),
                                      (8203, 1.0), (32767, 0.9), (32768, 0.74), (32768, 0.76), (65600, 0.2), (65600, 0.6),
                                      (65600, 0.9)])
def test_share_of_the_queries_in_a_crowd(n2, share, K):
    """Half of the points in one cell, and `share` of the queries beside them."""
    rng = np.random.default_rng(K)
    a = clouds("ball", 9)[0][:3000].copy()
    a[::2] = 0.3 + 1e-4 * rng.standard_normal((1500, 3))
    b = np.resize(clouds("surface", 9)[1], (n2, 3)) + 0.01 * rng.standard_normal((n2, 3))
    m = int(share * n2)
    b[rng.permutation(n2)[:m]] = 0.3 + 1e-4 * rng.standard_normal((m, 3))
    _check(a, b, K)


@pytest.mark.parametrize("n1,K", [(999, 4), (1000, 4), (1499, 1), (1500, 1), (599, 5), (600, 5), (299, 9), (300, 9), (300, 32)])
def test_sizes_from_which_the_grid_is_searched(n1, K):
    a, b = clouds("surface", 5)
    _check(a[:n1], b[:777], K)


@pytest.mark.parametrize("name", ["clusters", "same", "ball"])
def test_points_in_cell_order(name):
    a, b = clouds(name, 9)
    a = a[np.lexsort(np.floor(a.T * 8))]
    _check(a, b[:1000], 4)
