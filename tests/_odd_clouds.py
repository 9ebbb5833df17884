"""Clouds with points that are not finite, or so far (or so close) that their
squared distances over- or underflow, and the K nearest by key: (d2 bits, index)
in ascending order, infinite distances behind the finite ones and NaN behind
those."""
import numpy as np

from _grid_clouds import clouds

NAN, INF = np.float32(np.nan), np.float32(np.inf)
NAMES = ["nan", "nan coordinate", "inf", "far", "huge", "tiny", "nan axis", "inf axis", "all nan"]


def odd_cloud(name: str, n: int = 900, half: int = 0) -> np.ndarray:
    """n points; half = 1 gives another cloud of the same kind."""
    x = clouds("ball", 1 + n // 360)[half][:n].copy()
    assert len(x) == n
    p = [3 + half, n // 2, n - 2]
    if name == "nan":
        x[p[:2]] = NAN
    elif name == "nan coordinate":
        for a in range(3):
            x[p[a], a] = NAN
    elif name == "inf":
        x[p[0]] = [INF, INF, -INF]
        x[p[1], 0] = -INF
        x[p[2], 1] = INF
    elif name == "far":                    # finite; distances to it overflow
        x[p[0]] = 1e20
        x[p[1]] = [0.0, -2e19, 0.0]
    elif name == "huge":                   # about half of the distances overflow
        x *= np.float32(2e19)
    elif name == "tiny":                   # all distances underflow
        x *= np.float32(1e-24)
    elif name == "nan axis":
        x[:, 1] = NAN
    elif name == "inf axis":
        x[:, 2] = np.where(np.arange(n) % 3 == half, -INF, x[:, 2])
    else:
        assert name == "all nan", name
        x[:] = NAN
    return x


def distances(q, c) -> np.ndarray:
    """float32 squared distances, each operation rounded once."""
    with np.errstate(all="ignore"):
        d = q[:, None, :] - c[None]
        d = d * d
        return (d[..., 0] + d[..., 1]) + d[..., 2]


def nearest(q, c, K, skip_self=False):
    """(indices [n, K], -1 past the candidates; their squared distances, 0 past them)."""
    d = distances(q, c)
    assert not np.signbit(d[~np.isnan(d)]).any()
    key = np.where(np.isnan(d), np.float32(np.nan), d).astype(np.float32).view(np.uint32).astype(np.uint64)
    key = np.where(np.isnan(d), np.uint64(0x7FC00000), key) << np.uint64(32) | np.arange(len(c), dtype=np.uint64)
    keff = min(K, len(c) - int(skip_self))
    if skip_self:
        np.fill_diagonal(key, ~np.uint64(0))
    idx = np.argsort(key, 1, kind="stable")[:, :keff].astype(np.int32)
    out = np.full((len(q), K), -1, np.int32)
    d2 = np.zeros((len(q), K), np.float32)
    out[:, :keff], d2[:, :keff] = idx, np.take_along_axis(d, idx, 1)
    return out, d2


def mean_rows(rows, idx):
    """FP64 mean of rows[idx[i, :]] in that order, rounded to float32."""
    with np.errstate(all="ignore"):
        acc = np.zeros((len(idx),) + rows.shape[1:])
        for k in range(idx.shape[1]):
            acc += rows[idx[:, k]].astype(np.float64)
        return (acc / idx.shape[1]).astype(np.float32)


def same_values(a, b):
    """Equal, NaN where the other is NaN."""
    return np.array_equal(np.asarray(a), np.asarray(b), equal_nan=True)
