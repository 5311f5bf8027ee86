"""Lloyd iterations with the nearest centroid from the matrix cores: up to 256 centroids, both sides of the rule, all dimensions, ragged numbers of
vectors; vectors far from the origin (many are decided by direct distances), coinciding centroids, centroids and vectors that
are not numbers."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [4, 6, 8, 12, 16])
@pytest.mark.parametrize("nt,k", [(40_000, 32), (1, 256), (33_001, 33), (4100, 255), (63, 100), (33_000, 96), (40_064, 256)])
@pytest.mark.parametrize("kind", ["plain", "far", "same", "bad", "off"])
def test_assignment(D, nt, k, kind):
    import paper_1901_00275_amd as vlq

    rng = np.random.default_rng(D + nt + k)
    C = rng.normal(size=(k, D))
    X = rng.normal(size=(nt, D)) * 1.2
    if kind == "far":
        C, X = C + 300.0, X + 300.0
    elif kind == "same":
        C[k // 2:] = C[: k - k // 2]
    C, X = C.astype(np.float32), X.astype(np.float32)
    if kind == "bad":
        C[k // 3, 1] = np.nan
        C[k - 1, 0] = np.inf
        X[nt // 2, 2] = np.inf
    shift = 1 if kind == "off" else 0  # rows off their 16-byte boundaries
    buf, cb = torch.empty(nt * D + 1, device=DEV), torch.empty(k * D + 1, device=DEV)
    Xd, Cd = buf[shift:shift + nt * D].view(nt, D), cb[shift:shift + k * D].view(k, D)
    Xd.copy_(torch.as_tensor(X))
    Cd.copy_(torch.as_tensor(C))
    a, counts = torch.empty(nt, dtype=torch.int32, device=DEV), torch.empty(k, dtype=torch.int32, device=DEV)
    vlq.vlq_kmeans(Xd, nt, D, k, 0, Cd, a, counts)
    a = a.cpu().numpy()
    assert ((a >= 0) & (a < k)).all()
    assert np.array_equal(counts.cpu().numpy(), np.bincount(a, minlength=k))
    Xq, Cq = torch.as_tensor(X).to(DEV).double(), torch.as_tensor(C).to(DEV).double()
    for s in range(0, nt, 4096):
        d = ((Xq[s:s + 4096, None] - Cq[None]) ** 2).sum(2).cpu().numpy()
        d[~np.isfinite(d)] = np.inf
        fine = np.isfinite(d.min(1))
        got, best = d[np.arange(len(d)), a[s:s + 4096]], d.min(1)
        # the direct fp32 distances decide: D + 1 roundings in each of the two compared, and the rounding of the differences
        assert (got[fine] <= best[fine] * (1 + 2 * (D + 2) * 2.0 ** -24)).all()
        first = fine & (got == best)
        if kind == "same":
            assert np.array_equal(a[s:s + 4096][first], d.argmin(1)[first])
        assert (a[s:s + 4096][~fine] == 0).all()


def direct(X, C):
    """The direct distances in fp32, operation by operation (a product of two fp32 numbers is exact in fp64)."""
    f32, D = np.float32, X.shape[1]
    with np.errstate(over="ignore", invalid="ignore"):
        t = (X[:, None] - C[None]).astype(np.float64)
        q = 4 if D % 4 == 0 else 1
        v = []
        for p in range(0, D, q):
            acc = np.zeros(t.shape[:2], f32)
            for d in range(p, p + q):
                acc = (t[..., d] * t[..., d] + acc).astype(f32)
            v.append(acc)
        s = v[0] + v[1]
        for i in range(2, len(v), 2):
            s = s + (v[i] + v[i + 1] if i + 1 < len(v) else v[i])
    return s


def nearest(X, C):
    """The first centroid at the smallest direct distance; 0 where none is at a finite one."""
    a = []
    for s in range(0, len(X), 512):
        d = direct(X[s:s + 512], C)
        d[~np.isfinite(d)] = np.inf
        a.append(np.where(np.isfinite(d.min(1)), d.argmin(1), 0))
    return np.concatenate(a)


def assigned(X, C):
    import paper_1901_00275_amd as vlq

    nt, D = X.shape
    a = torch.empty(nt, dtype=torch.int32, device=DEV)
    vlq.vlq_kmeans(torch.as_tensor(X).to(DEV), nt, D, len(C), 0, torch.as_tensor(C).to(DEV), a, None)
    return a.cpu().numpy()


@pytest.mark.parametrize("D,k", [(6, 256), (8, 256), (12, 200), (16, 256), (16, 97)])
@pytest.mark.parametrize("kind", ["1e20", "1e23", "1e38", "beside"])
def test_norms_that_overflow(D, k, kind):
    """Finite centroids whose squared norms overflow fp32, and vectors beside one of them."""
    rng = np.random.default_rng(D + k)
    C, X = rng.normal(size=(k, D)), rng.normal(size=(2100, D)) * 1.2
    if kind == "beside":
        C[k // 3] = 3e19
        X[::7] = 3e19 * (1 + 1e-3 * rng.normal(size=X[::7].shape))
    else:
        C[k // 3, 1] = float(kind)
    C, X = C.astype(np.float32), X.astype(np.float32)
    want = nearest(X, C)
    assert len(np.unique(want)) > k // 2 and (kind != "beside" or (want[::7] == k // 3).all())
    assert np.array_equal(assigned(X, C), want)


@pytest.mark.parametrize("D,k", [(6, 256), (8, 200), (12, 200), (16, 256)])
@pytest.mark.parametrize("scale", [2.0 ** -72, 2.0 ** -68, 2.0 ** -64, 2.0 ** -61, 2.0 ** -57])
def test_squares_below_the_normal_range(D, k, scale):
    """Squared distances that fp32 holds with a few bits only: roundings no longer relative to the values."""
    rng = np.random.default_rng(D + k)
    C, X = (rng.normal(size=(k, D)) * scale).astype(np.float32), (rng.normal(size=(4100, D)) * 1.2 * scale).astype(np.float32)
    assert np.array_equal(assigned(X, C), nearest(X, C))


@pytest.mark.parametrize("D,k", [(6, 256), (8, 200), (12, 200), (16, 256), (16, 96)])
@pytest.mark.parametrize("far,times", [(1, 30.0), (1, 100.0), (1, 1e6), (1, 1e15), (30, 100.0), (200, 1e4), (3, -1.0)])
def test_far_centroids(D, k, far, times):
    """Centroids far from the others (times -1: all else in one point), and vectors near them, between and beyond."""
    rng = np.random.default_rng(D + k + far)
    C, X = rng.normal(size=(k, D)), rng.normal(size=(4100, D)) * 1.2
    if times < 0:
        C[far:] = C[k - 1] + 1e-3 * rng.normal(size=C[far:].shape)
    else:
        C[: min(far, k // 2)] *= times
    near = rng.integers(0, max(1, min(far, k // 2)), 600)
    X[:200] = C[near[:200]] * (1 + 1e-3 * rng.normal(size=(200, D)))
    X[200:400] = C[near[200:400]] * rng.uniform(0.45, 0.55, (200, 1))
    X[400:600] = C[near[400:600]] * rng.uniform(1, 3, (200, 1))
    C, X = C.astype(np.float32), X.astype(np.float32)
    assert np.array_equal(assigned(X, C), nearest(X, C))


def time_of(X, C, iters=0):
    import paper_1901_00275_amd as vlq

    best, a = np.inf, torch.empty(len(X), dtype=torch.int32, device=DEV)
    for _ in range(8):
        s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start = C.clone()
        torch.cuda.synchronize()
        s.record()
        vlq.vlq_kmeans(X, len(X), X.shape[1], len(C), iters, start, a, None)
        e.record()
        e.synchronize()
        best = min(best, s.elapsed_time(e))
    return best


def vectors():
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    return torch.randn(262_144, 16, generator=g, device=DEV)


def test_a_far_centroid_costs_nothing():
    """One centroid at 30 to 10^15 times the norm of the others: not every vector is compared with all centroids."""
    X = vectors()
    base = X[:256].clone()
    plain = time_of(X, base)
    for times in (30.0, 100.0, 1e6, 1e15):
        C = base.clone()
        C[77] *= times
        assert time_of(X, C) < 1.25 * plain, times


@pytest.mark.parametrize("kind", ["overflow", "coinciding"])
def test_codebooks_without_use_for_the_products(kind):
    """A centroid whose norm overflows, and one centroid 256 times: no slower than the walk alone, which takes 264 centroids."""
    X = vectors()
    C = X[:256].clone()
    if kind == "overflow":
        C[3] = 1e21
    else:
        C[:] = X[0]
    assert time_of(X, C) < 1.2 * time_of(X, X[:264].clone())


def tight_groups(D, k, nt):
    """Vectors in k / 4 groups that are far narrower than their distance from each other, so that the products decide nothing."""
    g = torch.Generator(device=DEV)
    g.manual_seed(D + k)
    X = 10 * torch.randn(k // 4, D, generator=g, device=DEV)[torch.randint(0, k // 4, (nt,), generator=g, device=DEV)]
    return X + 0.01 * torch.randn(nt, D, generator=g, device=DEV)


@pytest.mark.parametrize("D,k,nt", [(6, 256, 4100), (8, 255, 4100), (12, 128, 33_000), (16, 256, 4100)])
def test_iterations_of_one_call_and_of_many(D, k, nt):
    """The iterations that leave the products out give what those with them do."""
    import paper_1901_00275_amd as vlq

    X = tight_groups(D, k, nt)
    one, many = X[:k].clone(), X[:k].clone()
    assign, counts = torch.empty(nt, dtype=torch.int32, device=DEV), torch.empty(k, dtype=torch.int32, device=DEV)
    vlq.vlq_kmeans(X, nt, D, k, 7, one, assign, counts)
    for _ in range(7):
        vlq.vlq_kmeans(X, nt, D, k, 1, many, None, None)
    assert torch.equal(one, many)
    want = nearest(X.cpu().numpy(), many.cpu().numpy())
    assert np.array_equal(assign.cpu().numpy(), want)
    assert np.array_equal(counts.cpu().numpy(), np.bincount(want, minlength=k))


def test_groups_that_the_products_do_not_tell_apart():
    """256 centroids, which the products serve, against 257, which they do not."""
    X = tight_groups(8, 256, 262_144)
    assert time_of(X, X[:256], 10) < 1.3 * time_of(X, X[:257], 10)
