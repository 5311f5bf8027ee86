"""Nearest centroid through the fp16 product against fp64: edges of tiles, splits and row blocks, many centroids inside the
band (slots and whole splits are searched exactly), rows and centroids of very different sizes."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


def on_device(V, off):
    """V on the GPU, `off` floats behind a 16-byte boundary"""
    buf = torch.empty(V.size + off, device=DEV)
    t = buf[off:].view(V.shape)
    t.copy_(torch.as_tensor(V))
    return t


def assign(X, C, off=0):
    import paper_1901_00275_amd as vlq

    a = torch.empty(len(X), dtype=torch.int32, device=DEV)
    vlq.vlq_kmeans(on_device(X, off), len(X), X.shape[1], len(C), 0, on_device(C, off), a, None)
    return a.cpu().numpy()


@pytest.mark.parametrize("kind", ["real", "integer", "near", "same", "tiny", "far", "outlier"])
@pytest.mark.parametrize("nt,D,k", [(1, 128, 300), (127, 96, 1), (129, 32, 129), (1000, 64, 5000), (700, 128, 1024 + 33), (300, 96, 9000)])
def test_nearest_centroid(kind, nt, D, k):
    rng = np.random.default_rng(nt + k)
    C = rng.normal(size=(k, D))
    X = C[rng.integers(0, k, nt)] + rng.normal(scale=0.5, size=(nt, D))
    if kind == "integer":
        C, X = C * 40, np.rint(X * 40)
    elif kind == "near":  # all centroids within the product's error of each other
        C = C[:1] + rng.normal(scale=1e-4, size=(k, D))
    elif kind == "same":  # groups of coinciding centroids: the smaller index
        C = C[rng.integers(0, max(1, k // 40), k)]
    elif kind == "tiny":  # a centroid and a row that vanish beside the others
        C[k // 2] *= 1e-11
        X[nt // 2] *= 1e-11
    elif kind == "far":
        X[nt // 2] *= 1e7
    elif kind == "outlier":
        C[0] *= 1e5
    X, C = X.astype(np.float32), C.astype(np.float32)
    cell = assign(X, C)
    assert ((cell >= 0) & (cell < k)).all()
    for s in range(0, nt, 64):
        d = ((X[s:s + 64, None].astype(np.float64) - C[None]) ** 2).sum(2)
        got = d[np.arange(len(d)), cell[s:s + 64]]
        # fp32 direct distances decide: D + 1 roundings in each of the two compared
        assert (got <= d.min(1) * (1 + 2 * (D + 1) * 2.0 ** -24)).all()
        if kind == "same":
            exact = got == d.min(1)
            assert np.array_equal(cell[s:s + 64][exact], d.argmin(1)[exact])


def rows_apart(nt, D, k, seed=0):
    """Centroids and vectors of ordinary size, and a few vectors ten million times as large among them."""
    rng = np.random.default_rng(seed)
    C = rng.normal(size=(k, D))
    X = C[rng.integers(0, k, nt)] + rng.normal(scale=0.3, size=(nt, D))
    far = np.arange(5, nt, 211)
    X[far] *= 1e7
    return X.astype(np.float32), C.astype(np.float32), far


@pytest.mark.parametrize("nt,D,k", [(300, 128, 700), (1000, 32, 129), (128, 96, 4096), (129, 64, 1000)])
@pytest.mark.parametrize("kind", ["far", "spread", "lost"])
def test_rows_of_one_block_differ_in_size(kind, nt, D, k):
    X, C, far = rows_apart(nt, D, k)
    rng = np.random.default_rng(1)
    ok = np.ones(nt, bool)
    if kind == "spread":  # any size from 1e-6 to 1e6
        X *= (10.0 ** rng.uniform(-6, 6, (nt, 1))).astype(np.float32)
    elif kind == "lost":  # beside 1e23 the squares of the others vanish (and its own overflows: any cell will do)
        X[far] = 1e23
        X[~np.isin(np.arange(nt), far)] *= 1e-6
        C *= 1e-6
        ok[far] = False
    cell = assign(X, C)
    assert ((cell >= 0) & (cell < k)).all()
    X64, C64 = X.astype(np.float64), C.astype(np.float64)
    for i in np.flatnonzero(ok):
        d = ((X64[i] - C64) ** 2).sum(1)
        assert d[cell[i]] <= d.min() * (1 + 2 * (D + 1) * 2.0 ** -24), i


def time_assign(X, C):
    import paper_1901_00275_amd as vlq

    Xd, Cd = torch.as_tensor(X).to(DEV), torch.as_tensor(C).to(DEV)
    a = torch.empty(len(X), dtype=torch.int32, device=DEV)
    best = float("inf")
    for _ in range(4):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        vlq.vlq_kmeans(Xd, len(X), X.shape[1], len(C), 0, Cd, a, None)
        t1.record()
        t1.synchronize()
        best = min(best, t0.elapsed_time(t1))
    return best


def test_small_rows_beside_ordinary_ones_cost_nothing():
    """With one scale for a block, its small rows were lost and compared with every centroid one by one."""
    X, C, far = rows_apart(60_000, 128, 16_384)
    X[far] *= 1e-7
    ordinary = time_assign(X, C)
    X[::2] *= 1e-8
    assert time_assign(X, C) < 2 * ordinary


@pytest.mark.parametrize("off", [0, 1])
@pytest.mark.parametrize("nt,D,k,group,spread", [
    (1000, 128, 5000, 16, 0.04), (300, 96, 20_000, 64, 0.03), (129, 32, 3000, 250, 0.01), (70_000, 64, 2048, 40, 0.02), (3, 128, 9000, 3000, 0.001)])
def test_crowded_groups_of_centroids(nt, D, k, group, spread, off):
    """Tight groups of centroids (more of them inside the band than a shortlist holds), some coinciding, and vectors that
    are not numbers among the others."""
    rng = np.random.default_rng(k)
    C = np.repeat(rng.normal(size=(k // group + 1, D)), group, 0)[:k] + spread * rng.normal(size=(k, D))
    C[k // 2:k // 2 + 9] = C[7]
    X = C[rng.integers(0, k, nt)] + rng.normal(scale=0.3, size=(nt, D))
    X[nt // 3] = C[k // 2] + 1e-3
    X, C = X.astype(np.float32), C.astype(np.float32)
    bad = np.arange(1, nt, 97)
    X[bad, 3] = np.nan
    cell = assign(X, C, off)
    assert ((cell >= 0) & (cell < k)).all()
    Xd, Cd = torch.as_tensor(X).to(DEV).double(), torch.as_tensor(C).to(DEV).double()
    for s in range(0, nt, 64):
        d = ((Xd[s:s + 64, None] - Cd[None]) ** 2).sum(2).cpu().numpy()
        got = d[np.arange(len(d)), cell[s:s + 64]]
        fine = ~np.isnan(d[:, 0])
        assert (got[fine] <= d[fine].min(1) * (1 + 2 * (D + 1) * 2.0 ** -24)).all()
        first = fine & (got == d.min(1))
        assert np.array_equal(cell[s:s + 64][first], d.argmin(1)[first])


def test_crowded_codebooks_and_far_rows_take_no_more_than_a_second_product():
    """One wave read all centroids for every such vector: 28 times as long with groups of 16, 11 times with far rows."""
    rng = np.random.default_rng(3)
    nt, D, k = 131_072, 128, 16_384
    t = {}
    for spread in (0.3, 0.04, 0.001):
        C = np.repeat(rng.normal(size=(k // 16, D)), 16, 0) + spread * rng.normal(size=(k, D))
        X = C[rng.integers(0, k, nt)] + rng.normal(scale=0.3, size=(nt, D))
        t[spread] = time_assign(X.astype(np.float32), C.astype(np.float32))
    assert t[0.04] < 5 * t[0.3] and t[0.001] < 5 * t[0.3], t
    X, C, far = rows_apart(nt, D, k)
    with_far = time_assign(X, C)
    X[far] *= 1e-7
    assert with_far < 5 * time_assign(X, C)


@pytest.mark.parametrize("nt,k", [(130, 1), (130, 5), (300, 127), (130, 1300)])
def test_all_columns_read_exactly(nt, k):
    """Nothing separates the columns in fp16 (every row is compared with all of them): the smallest exact distance, the
    smaller index of a tie."""
    D = 64
    rng = np.random.default_rng(k)
    C = (1.0 + 1e-6 * rng.integers(-8, 9, (k, D))).astype(np.float32)
    C[k // 2:] = C[:k - k // 2]  # each twice
    X = (1000.0 + rng.integers(0, 3, (nt, D))).astype(np.float32)
    X[:, 0] += np.arange(nt)
    cell = assign(X, C)
    # the direct sum in the order of the kernel: four components per lane, then pairs of lanes
    t = X[:, None] - C[None]
    acc = np.zeros((nt, k, 16))
    for d in range(4):  # (fused: each step is rounded once, from a product that fp64 holds exactly)
        acc = (t[:, :, d::4].astype(np.float64) ** 2 + acc).astype(np.float32)
    for _ in range(4):
        acc = acc[..., 0::2] + acc[..., 1::2]
    assert acc.dtype == np.float32
    assert np.array_equal(cell, acc[..., 0].argmin(1))
