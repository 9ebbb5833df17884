"""Argument checks of dpr_topk_sh_ws and dpr_topk_sh_ws_bytes: on the host,
before anything is launched (the pointers are never read)."""
import pytest

FAKE = 0x10000000
INVALID, WORKSPACE = 1, 2


@pytest.fixture(scope="module")
def lib():
    from paper_2205_14330_amd import _abi
    return _abi.load()


@pytest.mark.parametrize("case,code", [("n1", INVALID), ("n2", INVALID), ("K0", INVALID), ("K33", INVALID),
                                       ("degree", INVALID), ("null_s1", INVALID), ("null_sh", INVALID),
                                       ("null_s2", INVALID), ("null_out", INVALID), ("null_ws", WORKSPACE),
                                       ("short_ws", WORKSPACE), ("misaligned_ws", INVALID)])
@pytest.mark.parametrize("n1", [100, 5000])                # by brute force, through the grid
def test_invalid_arguments_rejected(lib, n1, case, code):
    a = dict(n1=n1, s1=FAKE, sh=FAKE, n2=80, s2=FAKE, degree=2, K=4, out=FAKE, ws=FAKE,
             nb=lib.dpr_topk_sh_ws_bytes(n1, 80, 4))
    assert a["nb"] > 0
    a.update({"n1": dict(n1=0), "n2": dict(n2=-1), "K0": dict(K=0), "K33": dict(K=33), "degree": dict(degree=4),
              "null_s1": dict(s1=None), "null_sh": dict(sh=None), "null_s2": dict(s2=None), "null_out": dict(out=None),
              "null_ws": dict(ws=None), "short_ws": dict(nb=a["nb"] - 1), "misaligned_ws": dict(ws=FAKE + 8)}[case])
    rc = lib.dpr_topk_sh_ws(a["n1"], a["s1"], a["sh"], a["n2"], a["s2"], a["degree"], a["K"], a["out"], None, a["ws"],
                            a["nb"], None)
    assert rc == code and lib.dpr_last_error()


def test_workspace_bytes(lib):
    for n1, n2, K in ((0, 5, 4), (5, -1, 4), (5, 5, 0), (5, 5, 33), (1 << 31, 5, 4)):
        assert lib.dpr_topk_sh_ws_bytes(n1, n2, K) == 0
    for K in (1, 4, 8, 32):
        sizes = [lib.dpr_topk_sh_ws_bytes(n, 1000, K) for n in (1, 299, 300, 999, 1000, 100000)]
        assert sizes == sorted(sizes) and sizes[0] > 0
    assert lib.dpr_topk_sh_ws_bytes(5000, 0, 4) > 0
