"""CPU build of the grid searches of the video warm start under AddressSanitizer
and UndefinedBehaviorSanitizer, against the oracle: nearest and top-k indices
and the SH means bit for bit; Eq. (9) to 1e-12 (FP64 sums of about 10^3 terms
in another order); the gradient to float32 rounding."""
import os

import numpy as np
import pytest

import oracle
import workloads
from _grid_clouds import NAMES, clouds
from _hostbuild import compile_harness, run


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    return compile_harness("grid_host", tmp_path_factory.mktemp("hostbuild"))


def _read(d, name, dtype, shape):
    return np.fromfile(os.path.join(str(d), name), dtype).reshape(shape)


@pytest.mark.parametrize("name", NAMES)
def test_chamfer(exe, tmp_path, name):
    s1, s2 = clouds(name)
    run(exe, tmp_path, "chamfer", {"s1": s1, "s2": s2})
    assert np.array_equal(_read(tmp_path, "nn12.bin", np.int32, (-1,)), oracle.chamfer_nn(s1, s2)[0])
    assert np.array_equal(_read(tmp_path, "nn21.bin", np.int32, (-1,)), oracle.chamfer_nn(s2, s1)[0])
    rcd, rg = oracle.chamfer(s1, s2)
    assert float(_read(tmp_path, "cd.bin", np.float64, (1,))[0]) == pytest.approx(rcd, rel=1e-12, abs=1e-300)
    np.testing.assert_allclose(_read(tmp_path, "grad2.bin", np.float32, (-1, 3)), rg, rtol=1e-6,
                               atol=1e-7 * max(np.abs(rg).max(), 1e-30))


@pytest.mark.parametrize("name,K,deg", [("ball", 4, 2), ("surface", 1, 1), ("floaters", 8, 0), ("apart", 5, 2),
                                        ("clusters", 16, 1), ("duplicates", 12, 2), ("line", 9, 0), ("thin", 32, 3),
                                        ("same", 3, 1)])
def test_topk(exe, tmp_path, name, K, deg):
    s1, s2 = clouds(name)
    s2 = s2[:200]
    sh1 = workloads.point_attributes(len(s1), deg, K)[0]
    run(exe, tmp_path, "topk", {"s1": s1, "sh1": sh1, "s2": s2}, 3 * (deg + 1) ** 2, K)
    rout, ridx = oracle.topk_sh(s1, sh1, s2, K)
    assert np.array_equal(_read(tmp_path, "idx.bin", np.int32, (len(s2), K)), ridx)
    assert np.array_equal(_read(tmp_path, "out_sh.bin", np.float32, rout.shape), rout.astype(np.float32))


def test_topk_with_fewer_points_than_k(exe, tmp_path):
    s1, s2 = clouds("ball")
    s1 = s1[:5]
    sh1 = workloads.point_attributes(5, 2, 1)[0]
    run(exe, tmp_path, "topk", {"s1": s1, "sh1": sh1, "s2": s2}, 27, 8)
    rout, ridx = oracle.topk_sh(s1, sh1, s2, 8)
    assert np.array_equal(_read(tmp_path, "idx.bin", np.int32, (len(s2), 8)), ridx)
    assert np.array_equal(_read(tmp_path, "out_sh.bin", np.float32, rout.shape), rout.astype(np.float32))
