"""GPU parity of one k-means step (MR_MAP_KMEANS) against the float64 oracle.

Tolerances (float32 arithmetic on the GPU, float64 in the oracle):
* assignment a_i is accepted iff d64(a_i) <= d64_min * (1 + 1e-6) + 1e-12
  (ties within 1e-6 relative may go either way);
* counts are exact given the GPU's assignments;
* sums: |s32 - s64| <= 1e-5 * max(|s64|, sum_i |x_id|) per (cluster, dim),
  s64 recomputed in float64 with the GPU's assignments;
* centroids: new centroid = s / n in float64 rounded to float32, same bound
  divided by n.
"""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as t
    return t


def _run(torch, X, Cn, offset=0):
    from paper_1309_0215_amd import Job
    job = Job(device=0, km_centroids=torch.from_numpy(Cn).to("cuda:0"))
    Xd = torch.from_numpy(X).to("cuda:0")
    if offset:
        big = torch.zeros(X.size + offset, dtype=torch.float32, device="cuda:0")
        big[offset:] = Xd.reshape(-1)
        Xd = big[offset:].view(X.shape)
    a, s, c, cent, st = job.kmeans(Xd)
    return (a.cpu().numpy(), s.cpu().numpy(), c.cpu().numpy().view(np.uint32), cent.cpu().numpy(), st)


def _check_assign(X, Cn, a, idx=None):
    if idx is None:
        idx = np.arange(len(X))
    D = oracle.kmeans_distances(X[idx], Cn)
    dmin = D.min(axis=1)
    dg = D[np.arange(len(idx)), a[idx]]
    ok = dg <= dmin * (1 + 1e-6) + 1e-12
    assert ok.all(), (np.flatnonzero(~ok)[:10], dg[~ok][:5], dmin[~ok][:5])
    return int((a[idx] != D.argmin(axis=1)).sum())


def _check_assign_all(X, Cn, a, chunk=1 << 20):
    """_check_assign over every point, for sizes where the direct form of
    every distance takes minutes. Each point is screened with the expanded
    float64 form |x|^2 - 2 x.c + |c|^2 (float32 inputs: the products are
    exact, the 32-term sums round by less than 32 * 2^-53 of |x|^2 + 2|x||c|
    + |c|^2), taken here with the margin m = 1e-12 (|x|^2 + max |c|^2), over
    a hundred times that bound. A point whose distance to its assigned
    centroid lies more than 3m inside the acceptance limit passes, more than
    3m outside it fails; the others are decided by the oracle's direct form.
    Returns the number of points so decided."""
    C64 = np.asarray(Cn, np.float64)
    cn = (C64 * C64).sum(axis=1)
    near = []
    for lo in range(0, len(X), chunk):
        x = np.asarray(X[lo:lo + chunk], np.float64)
        xn = (x * x).sum(axis=1)
        De = xn[:, None] - 2.0 * (x @ C64.T) + cn[None, :]
        lim = De.min(axis=1) * (1 + 1e-6) + 1e-12
        dg = De[np.arange(len(x)), a[lo:lo + chunk]]
        m = 1e-12 * (xn + cn.max())
        assert not (dg > lim + 3 * m).any(), lo + np.flatnonzero(dg > lim + 3 * m)[:10]
        near.append(lo + np.flatnonzero(np.abs(dg - lim) <= 3 * m))
    idx = np.concatenate(near)
    if len(idx):
        _check_assign(X, Cn, a, idx)
    return len(idx)


def _check_update(X, Cn, a, s, c, cent):
    k = len(Cn)
    S64, n64, newC = oracle.kmeans_update(X, a, Cn)
    assert np.array_equal(c.astype(np.int64), n64)
    A = oracle.kmeans_abs_sums(X, a, k)
    tol = 1e-5 * np.maximum(np.abs(S64), A)
    assert (np.abs(s.astype(np.float64) - S64) <= tol).all()
    ctol = tol / np.maximum(n64, 1)[:, None] + 1e-7 * np.abs(newC)
    assert (np.abs(cent.astype(np.float64) - newC) <= ctol).all()


@pytest.mark.parametrize("n", [1, 31, 32, 33, 4097, 50_000])
def test_mfma_path(torch, n):
    X, Cn = gen.kmeans(3, n=max(n, 64), d=32, k=64)
    X = X[:n].copy()
    a, s, c, cent, st = _run(torch, X, Cn)
    assert st["strategy_used"] == 1  # matrix-core path
    _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, c, cent)


@pytest.mark.parametrize("scale", [1e-3, 1e3])
def test_mfma_path_scales(torch, scale):
    # the near-tie bound scales with |x| and max |c|: small and large coordinates
    X, Cn = gen.kmeans(7, n=50_000, d=32, k=64)
    X = (X * scale).astype(np.float32)
    Cn = (Cn * scale).astype(np.float32)
    a, s, c, cent, st = _run(torch, X, Cn)
    assert st["strategy_used"] == 1
    _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, c, cent)


def test_tiny_coordinates_redo_the_step_generically(torch):
    # a nonzero coordinate below 2^-100 (in a point or a centroid) is outside
    # the exact bfloat16 split of the matrix-core path: the generic kernel
    # redoes the step
    X, Cn = gen.kmeans(8, n=4096, d=32, k=64)
    X = X.copy()
    X[100:200] *= np.float32(1e-33)
    a, s, c, cent, st = _run(torch, X, Cn)
    assert st["strategy_used"] == 0
    _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, c, cent)
    X, Cn = gen.kmeans(9, n=4096, d=32, k=64)
    Cn = Cn.copy()
    Cn[5, 3] = np.float32(1e-35)
    a, s, c, cent, st = _run(torch, X, Cn)
    assert st["strategy_used"] == 0
    _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, c, cent)


def test_generic_path_any_shape(torch):
    rng = np.random.default_rng(2)
    X = rng.standard_normal((3001, 5)).astype(np.float32)
    Cn = X[:7].copy()
    a, s, c, cent, st = _run(torch, X, Cn)
    assert st["strategy_used"] == 0
    _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, c, cent)


# the generic path's edges: one block of 32 centroids and one past it, four
# blocks and one past them; dims around the 8-dim chunk, the widest rows that
# share a workgroup (120) and one past them, the widest of all; cluster
# counts whose sums fill one LDS slice, and several (1024 x 17, 1024 x 256)
@pytest.mark.parametrize("n,d,k,shift", [
    (1, 1, 1, 0), (33, 1, 2, 0), (31, 7, 32, 0), (97, 8, 33, 0), (1500, 9, 3, 1000), (700, 12, 64, 0),
    (513, 16, 65, 0), (1025, 33, 128, 0), (260, 64, 129, 1000), (200, 120, 40, 0), (200, 121, 40, 0),
    (4100, 17, 1024, 0), (3000, 255, 5, 0), (2100, 256, 1024, 0)])
def test_generic_path_edges(torch, n, d, k, shift):
    """Random points and centroids drawn apart; `shift` adds a common offset,
    which puts every score gap within the float32 rounding bound."""
    rng = np.random.default_rng(n + d + k)
    X = (rng.standard_normal((n, d)) + shift).astype(np.float32)
    Cn = (rng.standard_normal((k, d)) + shift).astype(np.float32)
    for offset in (0, 1):
        a, s, c, cent, st = _run(torch, X, Cn, offset=offset)
        assert st["strategy_used"] == 0
        _check_assign(X, Cn, a)
        _check_update(X, Cn, a, s, c, cent)


def test_unaligned_points_use_generic_path(torch):
    X, Cn = gen.kmeans(4, n=2000, d=32, k=64)
    a, s, c, cent, st = _run(torch, X, Cn, offset=1)
    assert st["strategy_used"] == 0
    _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, c, cent)


def test_exact_ties_take_lowest_index_and_empty_clusters_keep_centroid(torch):
    X, Cn = gen.kmeans(5, n=8192, d=32, k=64)
    Cn = Cn.copy()
    Cn[10] = Cn[3]          # identical centroids: every point of cluster 3 ties with 10
    Cn[20] = 1000.0         # far away: an empty cluster
    a, s, c, cent, st = _run(torch, X, Cn)
    assert not (a == 10).any() and not (a == 20).any()
    assert c[20] == 0 and np.array_equal(cent[20], Cn[20])
    _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, c, cent)


def test_points_equal_to_centroids(torch):
    X, Cn = gen.kmeans(6, n=64, d=32, k=64)
    a, s, c, cent, st = _run(torch, Cn.copy(), Cn)
    assert np.array_equal(a, np.arange(64))


@pytest.mark.parametrize("d,k", [(32, 64), (5, 7)])
def test_no_points(torch, d, k):
    """An input of no points: every cluster is empty, so the counts and sums
    are zero and every centroid stays where it was (the oracle's update of an
    empty input gives the same)."""
    rng = np.random.default_rng(8)
    Cn = rng.standard_normal((k, d)).astype(np.float32)
    X = np.zeros((0, d), np.float32)
    a, s, c, cent, st = _run(torch, X, Cn)
    assert len(a) == 0 and (c == 0).all() and (s == 0).all()
    assert np.array_equal(cent, Cn)
    _check_update(X, Cn, a, s, c, cent)


def test_full_config_16m(torch):
    """The full 16,777,216-point step. The assignments of all points are
    checked (the first and the last 2^19, which hold the grid's ragged tail,
    against the oracle's direct form; every point through _check_assign_all),
    the counts and sums over all points."""
    X, Cn = gen.kmeans(3)  # 16,777,216 x 32, k = 64, first 64 points
    a, s, c, cent, st = _run(torch, X, Cn)
    assert int(c.astype(np.int64).sum()) == len(X)
    half = 1 << 19
    idx = np.concatenate([np.arange(half), np.arange(len(X) - half, len(X))])
    _check_assign(X, Cn, a, idx)
    print(f"points decided by the direct form: {_check_assign_all(X, Cn, a)}")
    # sums over all points in float64 with the GPU's assignments (bincount per dim)
    k, d = Cn.shape
    n64 = np.bincount(a, minlength=k)
    assert np.array_equal(c.astype(np.int64), n64)
    worst_rel = 0.0
    for t in range(d):
        col = X[:, t].astype(np.float64)
        S = np.bincount(a, weights=col, minlength=k)
        A = np.bincount(a, weights=np.abs(col), minlength=k)
        err = np.abs(s[:, t].astype(np.float64) - S)
        assert (err <= 1e-5 * np.maximum(np.abs(S), A)).all()
        # the plain relative bound wherever the sum is not a cancellation
        big = np.abs(S) > 1e-3 * A
        assert (err[big] <= 1e-5 * np.abs(S[big])).all()
        worst_rel = max(worst_rel, float((err[big] / np.abs(S[big])).max(initial=0.0)))
    print(f"largest plain relative sum error {worst_rel:.3e}")
    assert st["km_rechecked"] < len(X) // 100


# d = 32, k = 64 around a workgroup's twelve groups of 32 points, one and two
# passes of 256 workgroups, with what its rules turn on: zeros among the
# coordinates, points midway between two centroids (decided in float64), equal
# centroids (the lowest index), scores of both signs and of any size
@pytest.mark.parametrize("n,kind", [
    (383, "zeros"), (384, "ties"), (385, "ties"), (98_304, "zeros"), (98_305, "far"), (200_003, "ties"), (150_000, "near"),
])
def test_mfma_path_edges(torch, n, kind):
    rng = np.random.default_rng(n)
    Cn = rng.normal(size=(64, 32)).astype(np.float32)
    X = (Cn[rng.integers(0, 64, n)] + rng.normal(size=(n, 32)) * 0.3).astype(np.float32)
    if kind == "zeros":
        X[rng.random(X.shape) < 0.7] = 0.0
        Cn[rng.random(Cn.shape) < 0.5] = 0.0
    elif kind == "ties":
        Cn[40:] = Cn[:24]
        Cn = np.round(Cn * 8) / 8
        i, j = rng.integers(0, 64, n), rng.integers(0, 64, n)
        X = ((Cn[i] + Cn[j]) / 2).astype(np.float32)  # exact
    elif kind == "far":  # a common offset: norms far above the distances
        Cn += 100.0
        X += 100.0
    else:  # centroids within float32 rounding of each other
        Cn = (Cn[:1] + rng.normal(size=(64, 32)) * 1e-6).astype(np.float32)
        X = (Cn[:1] + rng.normal(size=(n, 32)) * 1e-3).astype(np.float32)
    a, s, c, cent, st = _run(torch, X, Cn)
    assert st["strategy_used"] == 1  # the matrix-core path
    if kind == "ties":
        assert np.array_equal(a, oracle.kmeans_distances(X, Cn).argmin(axis=1))
    else:
        _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, c, cent)


def test_mfma_path_points_that_are_no_numbers(torch):
    """The other points keep their clusters and the counts leave such points out."""
    rng = np.random.default_rng(5)
    Cn = rng.normal(size=(64, 32)).astype(np.float32)
    X = (Cn[rng.integers(0, 64, 5_000)] + rng.normal(size=(5_000, 32)) * 0.3).astype(np.float32)
    bad = np.arange(17, 5_000, 97)
    X[bad, bad % 32] = np.where(bad % 2, np.nan, np.inf)
    a, s, c, cent, st = _run(torch, X, Cn)
    ok = np.setdiff1d(np.arange(5_000), bad)
    _check_assign(X, Cn, a, ok)
    assert np.array_equal(c, np.bincount(a[ok], minlength=64) + np.bincount(a[bad][a[bad] < 64], minlength=64))


# caller workspaces that hold one partial but not the packed centroids (few
# dimensions, or few clusters): a thread per point decides in float64
@pytest.mark.parametrize("n,d,k", [(1, 1, 1), (1_000, 2, 64), (5_001, 3, 1024), (777, 256, 2), (20_000, 5, 7)])
def test_smallest_workspaces(torch, n, d, k):
    from paper_1309_0215_amd import Job
    X, Cn = gen.kmeans(n, n=max(n, k), d=d, k=k)
    X = X[:n].copy()
    up = lambda b: (b + 255) // 256 * 256
    ws = torch.empty(up(4 * k * d) + 512 + up(8 * k * d) + 4 * k, dtype=torch.uint8, device="cuda:0")
    job = Job(device=0, km_centroids=torch.from_numpy(Cn).to("cuda:0"), workspace=ws)
    for _ in range(2):
        a, s, c, cent, st = job.kmeans(torch.from_numpy(X).to("cuda:0"))
        assert st["device_allocs"] == 0
        a, s, c, cent = a.cpu().numpy(), s.cpu().numpy(), c.cpu().numpy().view(np.uint32), cent.cpu().numpy()
        _check_assign(X, Cn, a)
        _check_update(X, Cn, a, s, c, cent)


def _signed(rng, shape, lo, hi):
    """Magnitudes uniform in [lo, hi), either sign."""
    return (rng.uniform(lo, hi, shape) * rng.choice([-1.0, 1.0], shape)).astype(np.float32)


# Where squares and products leave float32 at its lower end, every point is
# decided in float64: the assignments are the oracle's, the lowest index on
# equal distances. (Magnitudes within a factor of two, so that none is below
# 2^-100, from where on the step is not the matrix-core path's. Distances drawn
# at random differ by far more than the 32 roundings of 2^-53 they are summed
# with.)
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("scale", [0.0, 1e-15, 1e-17, 1e-18, 1e-19, 1e-20, 1e-22, 1e-25, 1e-29])
def test_underflow_of_squares_and_products(torch, scale, offset):
    """scale 0: all centroids zero and ordinary points, so that every centroid
    is as near as any other."""
    rng = np.random.default_rng(11)
    Cn = _signed(rng, (64, 32), scale, 2 * scale)
    X = _signed(rng, (5_003, 32), scale or 1.0, 2 * (scale or 1.0))
    X[-64:] = Cn
    a, s, c, cent, st = _run(torch, X, Cn, offset=offset)
    assert st["strategy_used"] == (0 if offset else 1)
    assert np.array_equal(a, oracle.kmeans_distances(X, Cn).argmin(axis=1))
    _check_update(X, Cn, a, s, c, cent)


# The same at float32's upper end: |c|^2 past it, or the products alone. (Where
# points are far longer than centroids, all distances round to |x|^2 and the
# nearest centroid is any within the acceptance limit.)
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("x,c", [(1.0, 1e18), (1.0, 1e19), (1.0, 1e20), (1e18, 1e18), (1e20, 1e20), (1e20, 1.0), (1e30, 1e10),
                                 (1e10, 1e30), (1e33, 1e33)])
def test_overflow_of_squares_and_products(torch, x, c, offset):
    rng = np.random.default_rng(12)
    Cn = _signed(rng, (64, 32), c, 2 * c)
    X = _signed(rng, (5_003, 32), x, 2 * x)
    X[-64:] = Cn
    a, s, n, cent, st = _run(torch, X, Cn, offset=offset)
    assert st["strategy_used"] == (0 if offset else 1)
    if x <= c:
        assert np.array_equal(a, oracle.kmeans_distances(X, Cn).argmin(axis=1))
    else:
        assert a.min() >= 0 and a.max() < 64
        _check_assign(X, Cn, a)
    _check_update(X, Cn, a, s, n, cent)
