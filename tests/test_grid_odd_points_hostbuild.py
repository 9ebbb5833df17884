"""CPU build (AddressSanitizer, UndefinedBehaviorSanitizer) of the grid searches
on points that are not finite or whose distances over- or underflow: K valid
neighbours for every query, in the order of the keys, and a complete update."""
import numpy as np
import pytest

import oracle
import workloads
from _grid_clouds import clouds
from _hostbuild import compile_harness, run
from _odd_clouds import NAMES, mean_rows, nearest, odd_cloud, same_values


@pytest.fixture(scope="module")
def grid(tmp_path_factory):
    return compile_harness("grid_host", tmp_path_factory.mktemp("hostbuild"))


@pytest.fixture(scope="module")
def brute(tmp_path_factory):
    return compile_harness("chamfer_host", tmp_path_factory.mktemp("hostbuild"))


@pytest.fixture(scope="module")
def hybrid(tmp_path_factory):
    return compile_harness("hybrid_host", tmp_path_factory.mktemp("hostbuild"))


def _read(d, name, dtype, shape):
    return np.fromfile(str(d / name), dtype).reshape(shape)


@pytest.mark.parametrize("name,K", [(n, 1 + 4 * (i % 2)) for i, n in enumerate(NAMES)] + [("nan", 5), ("far", 5)])
def test_knn(hybrid, tmp_path, name, K):
    x = odd_cloud(name, 150)
    run(hybrid, tmp_path, "knn", {"xyz": x}, K)
    idx, d2 = nearest(x, x, K, skip_self=True)
    assert np.array_equal(_read(tmp_path, "idx.bin", np.int32, (-1, K)), idx)
    assert same_values(_read(tmp_path, "d2.bin", np.float32, (-1, K)), d2)


@pytest.mark.parametrize("name,K,odd", [(n, 1 + 3 * (i % 2), ("queries", "both")[i % 2]) for i, n in enumerate(NAMES)] +
                         [("nan", 4, "queries"), ("nan", 1, "points"), ("far", 4, "queries"), ("far", 1, "points"),
                          ("inf", 4, "queries"), ("inf", 1, "points"), ("nan coordinate", 4, "points")])
def test_topk(grid, tmp_path, name, K, odd):
    a = clouds("ball")[0][:200] if odd == "queries" else odd_cloud(name, 200)
    b = clouds("ball")[1][:12] if odd == "points" else odd_cloud(name, 12, 1)
    sh = workloads.point_attributes(len(a), 1, K)[0]
    run(grid, tmp_path, "topk", {"s1": a, "sh1": sh, "s2": b}, 12, K)
    idx, _ = nearest(b, a, K)
    assert np.array_equal(_read(tmp_path, "idx.bin", np.int32, (-1, K)), idx)
    assert np.array_equal(_read(tmp_path, "out_sh.bin", np.float32, (-1, 4, 3)), mean_rows(sh, idx))


@pytest.mark.parametrize("name,odd", [(n, ("s1", "s2", "both")[i % 3]) for i, n in enumerate(NAMES)] +
                         [("nan coordinate", "s1"), ("inf", "s1"), ("inf", "s2"), ("far", "both"), ("nan", "s2")])
def test_chamfer(grid, brute, tmp_path, name, odd):
    """Through the grid and by brute force: a point at no finite distance of any other has no nearest (-1); it takes
    part in no other point's gradient."""
    s1 = clouds("ball")[0][:160] if odd == "s2" else odd_cloud(name, 160)
    s2 = clouds("ball")[1][:150] if odd == "s1" else odd_cloud(name, 150, 1)
    n12, n21, cd, g = _eq9(s1, s2)
    for exe in (grid, brute):
        run(exe, tmp_path, "chamfer", {"s1": s1, "s2": s2})
        assert np.array_equal(_read(tmp_path, "nn12.bin", np.int32, (-1,)), n12)
        assert np.array_equal(_read(tmp_path, "nn21.bin", np.int32, (-1,)), n21)
        np.testing.assert_allclose(_read(tmp_path, "cd.bin", np.float64, (1,))[0], cd, rtol=1e-12)
        # rounding of FP64 sums in another order, then float32
        np.testing.assert_allclose(_read(tmp_path, "grad2.bin", np.float32, (-1, 3)), g, rtol=1e-6,
                                   atol=1e-7 * np.nanmax(np.abs(np.where(np.isfinite(g), g, 0.0))))


def _eq9(s1, s2):
    """nn12, nn21, Eq. (9) and its gradient, FP64."""
    def nn(q, c):
        i, d = nearest(q, c, 1)
        return np.where(d[:, 0] < np.inf, i[:, 0], -1), np.where(d[:, 0] < np.inf, d[:, 0], np.nan).astype(np.float64)
    (n12, d12), (n21, d21) = nn(s1, s2), nn(s2, s1)
    a, b = s1.astype(np.float64), s2.astype(np.float64)
    with np.errstate(all="ignore"):
        g = 2.0 / len(b) * (b - np.where(n21[:, None] >= 0, a[n21], np.nan))
        for i in np.nonzero(n12 >= 0)[0]:
            g[n12[i]] += 2.0 / len(a) * (b[n12[i]] - a[i])
        cd = d12.sum() / len(a) + d21.sum() / len(b)
    return n12, n21, cd, g


def _update(red, K, eps):
    """Steps 2 and 3 of Alg. 1 with neighbours by key: kept flags and the output rows."""
    f = np.float32
    idx, d2 = nearest(red[0], red[0], K, skip_self=True)
    with np.errstate(all="ignore"):
        d, s, v = np.sqrt(d2), np.zeros(len(d2), f), np.zeros(len(d2), f)
        for k in range(K):
            s = s + d[:, k]
        for k in range(K):
            v = v + (d[:, k] - s / f(K)) * (d[:, k] - s / f(K))
        keep = ~(np.sqrt(v / f(K)) > f(eps))
    kept = [a[keep] for a in red]
    idx, _ = nearest(kept[0], kept[0], K, skip_self=True)
    return keep, [np.concatenate([a, mean_rows(a, idx)]) for a in kept]


@pytest.mark.parametrize("name,share", [("nan", 0.02), ("nan coordinate", 0.02), ("nan coordinate", 0.3)])
def test_update(hybrid, tmp_path, name, share):
    """With few points removed (their neighbours renumbered) and many (a new search)."""
    K, N = 4, 64
    x = odd_cloud(name, 250)
    c = oracle.Cloud(x, *workloads.point_attributes(len(x), 1, 3))
    arrays = {"xyz": c.xyz, "sh": c.sh, "op": c.opacity, "rad": c.radius}
    arrays = {k: np.asarray(v, np.float32) for k, v in arrays.items()}
    run(hybrid, tmp_path, "voxel", arrays, N, 12)
    m = int(open(tmp_path / "counts.txt").read())
    red = [_read(tmp_path, f"out_{k}.bin", np.float32, s)[:m]
           for k, s in (("xyz", (-1, 3)), ("sh", (-1, 4, 3)), ("op", (-1,)), ("rad", (-1,)))]
    _, d2 = nearest(red[0], red[0], K, skip_self=True)
    s = np.sqrt(d2.astype(np.float64)).std(1)
    s = np.sort(s[np.isfinite(s)])
    eps = float(np.float32(s[int(len(s) * (1.0 - share))]))
    keep, want = _update(red, K, eps)
    assert 0 < (~keep).sum() < m // 2 and ((~keep).sum() <= m // 16) == (share < 0.05)
    run(hybrid, tmp_path, "hybrid", arrays, N, K, repr(eps), 12)
    counts = [int(v) for v in open(tmp_path / "counts.txt").read().split()]
    assert counts == [m, int(keep.sum()), 2 * int(keep.sum())]
    for k, w in zip(("xyz", "sh", "op", "rad"), want):
        assert same_values(_read(tmp_path, f"out_{k}.bin", np.float32, w.shape), w), k
