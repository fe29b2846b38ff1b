"""gorio_cluster_order against a plain numpy run of its stated rule: scores
summed in dimension order in float32, ties to the smaller centroid, means in
float64 (16 node ranges, members in id order), clusters' nodes in id order.
All of it is exact, so both must agree in every bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def plain(x, K, iterations):
    n, D = x.shape
    xf = x.astype(np.float32)
    c = xf[np.arange(K, dtype=np.int64) * n // K].copy()
    for it in range(iterations + 1):
        cc = np.zeros(K, np.float32)
        dot = np.zeros((n, K), np.float32)
        with np.errstate(all="ignore"):
            for d in range(D):
                cc = cc + c[:, d] * c[:, d]
                dot = dot + xf[:, d:d + 1] * c[None, :, d]
            s = cc[None, :] - np.float32(2) * dot
        key = np.zeros(n, np.int64)
        best = s[:, 0].copy()
        for k in range(1, K):
            less = s[:, k] < best
            best[less], key[less] = s[less, k], k
        if it == iterations:
            break
        for k in range(K):
            total, cnt = np.zeros(D), 0
            for t in range(16):
                m = np.nonzero(key[n * t // 16:n * (t + 1) // 16] == k)[0] + n * t // 16
                part = np.zeros(D)
                if len(m):
                    part = np.add.accumulate(x[m].astype(np.float64), axis=0)[-1]
                total, cnt = total + part, cnt + len(m)
            if cnt:
                c[k] = (total / cnt).astype(np.float32)
    order = np.argsort(key, kind="stable")
    n2s = np.empty(n, np.uint32)
    n2s[order] = np.arange(n, dtype=np.uint32)
    return n2s, c


def data(kind, n, D, seed):
    rng = np.random.default_rng(seed)
    lab = rng.integers(0, 12, n)
    if kind in ("same", "skew8"):   # all, or nearly all, rows the same: one cluster holds them
        x = rng.integers(0, 256, (n, D)).astype(np.uint8)
        x[rng.random(n) < (2.0 if kind == "same" else 0.97)] = x[0]
        return x
    if kind == "u8":
        return np.clip(np.rint(rng.uniform(40, 215, (12, D))[lab] + 20 * rng.standard_normal((n, D))), 0, 255).astype(np.uint8)
    if kind == "equal":      # few distinct rows: most scores tie exactly
        return rng.integers(0, 3, (7, D)).astype(np.uint8)[rng.integers(0, 7, n)]
    x = (rng.standard_normal((12, D))[lab] + 0.05 * rng.standard_normal((n, D))).astype(np.float32)
    if kind == "skew":       # one cluster holds nearly all rows
        x[rng.random(n) < 0.97] = x[0] + np.float32(0.25)
        x[::2] += np.float32(1e-3) * rng.standard_normal((len(x[::2]), D)).astype(np.float32)
    elif kind == "far":      # a large common offset: every score within rounding of the others
        x += np.float32(3000)
    elif kind == "nan":
        x[5, 0] = np.nan     # a row that is no initial centroid
        x[77, D - 1] = np.inf
    return x


@pytest.mark.parametrize("kind,n,D,K,iterations", [
    ("u8", 16384, 128, 32, 2),       # smallest batch and fewest centroids of the matrix path
    ("u8", 16383, 128, 32, 1),       # one vector fewer: the plain kernel
    ("u8", 20001, 100, 33, 2),       # one centroid past a tile, padded dimensions
    ("u8", 16500, 6, 40, 1),         # D no multiple of four
    ("f32", 16417, 96, 64, 2),
    ("f32", 17000, 17, 95, 2),
    ("f32", 16400, 129, 48, 1),      # one vector tile per wave
    ("f32", 16400, 256, 48, 1),
    ("f32", 16400, 257, 32, 1),      # past the matrix path's dimensions
    ("equal", 16390, 64, 50, 2),
    ("same", 16390, 128, 40, 2),     # every centroid repeats the first
    ("skew8", 20000, 100, 33, 2),
    ("skew8", 5001, 6, 9, 2),
    ("skew8", 1500, 1023, 3, 1),     # a row over more threads than a block has
    ("u8", 1025, 1024, 4, 1),        # one row past a block's share
    ("skew", 17000, 96, 33, 2),      # ranges of a thousand members, no multiple of the rows in flight
    ("skew", 40000, 300, 5, 2),
    ("f32", 513, 70, 16, 2),         # ranges of no, one or two members
    ("far", 16390, 96, 40, 1),
    ("nan", 16390, 96, 40, 0),
    ("f32", 3, 5, 3, 1),
])
def test_cluster_order_is_the_stated_rule(kind, n, D, K, iterations):
    import torch
    assert torch.cuda.is_available()   # before the library: both then share one HIP runtime
    import paper_2607_04415_amd as g
    x = data(kind, n, D, n + D)
    n2s, c = g.cluster_order(x, K, iterations)
    want_n2s, want_c = plain(x, K, iterations)
    assert np.array_equal(np.asarray(n2s, np.uint32), want_n2s)
    assert np.array_equal(np.asarray(c), want_c)
