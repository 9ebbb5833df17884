"""Pairs of clouds that stress the grid search: what decides its cell size, its
one-thread walk, the growing cube of the left-over queries and the brute-force
fall-back."""
import numpy as np


def _ball(rng, n):
    d = rng.standard_normal((n, 3))
    return d / np.linalg.norm(d, axis=1, keepdims=True) * rng.random((n, 1)) ** (1.0 / 3.0)


def clouds(name: str, scale: int = 1):
    """(s1, s2), float32."""
    rng = np.random.default_rng([7, len(name), ord(name[0])])
    n = 400 * scale
    a = _ball(rng, n)
    b = a[: n - 37] + 0.05 * rng.standard_normal((n - 37, 3))
    if name == "surface":                  # points on a sheet: few occupied cells
        a = rng.uniform(-1, 1, (n, 3))
        a[:, 2] = 0.3 * np.sin(3 * a[:, 0]) * np.cos(2 * a[:, 1])
        b = a[::-1] + 0.01 * rng.standard_normal((n, 3))
    elif name == "floaters":               # a few points far from everything stretch the box
        a[:7] *= 40.0
        b[:5] = -30.0 * b[:5]
    elif name == "apart":                  # disjoint clouds: every query is left over
        b = b + [9.0, 0.0, 0.0]
    elif name == "clusters":               # tight clusters: crowded cells
        c = rng.uniform(-1, 1, (3, 3))
        a = c[rng.integers(3, size=n)] + 1e-3 * rng.standard_normal((n, 3))
        b = c[rng.integers(3, size=n)] + 1e-3 * rng.standard_normal((n, 3))
        b[:9] = rng.uniform(-2, 2, (9, 3))
    elif name == "duplicates":             # coincident points and exact ties
        a = np.round(a * 4) / 4
        b = np.round(b * 4) / 4
    elif name == "flat":
        a[:, 1] = b[:, 1] = 0.125
    elif name == "line":
        a = np.outer(np.arange(n), [0.0, 0.0, 1.0])
        b = np.outer(np.arange(n - 50) + 0.5, [0.0, 0.0, 1.0])
    elif name == "one":                    # a single candidate
        b = b[:1]
    elif name == "same":                   # every point the same
        a[:] = a[0]
        b[:] = a[0]
    elif name == "far origin":             # cells are small against the coordinates
        a, b = a + 1000.0, b + 1000.0
    elif name == "thin":                   # an axis shorter than a cell
        a[:, 2] *= 1e-4
        b[:, 2] *= 1e-4
    else:
        assert name == "ball", name
    return a.astype(np.float32), b.astype(np.float32)


NAMES = ["ball", "surface", "floaters", "apart", "clusters", "duplicates", "flat", "line", "one", "same", "far origin",
         "thin"]
