"""Nearest centroid: strips of two row blocks (one or both present, last rows), odd and even numbers of column tiles, rows
whose scale is too far from the columns' for the norm to go into the products, centroids whose norm overflows."""
import numpy as np
import pytest
import torch

from test_gpu_nearest_half import assign
from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


def check(X, C, cell):
    X, C = X.astype(np.float64), C.astype(np.float64)
    for s in range(0, len(X), 64):
        d = ((X[s:s + 64, None] - C[None]) ** 2).sum(2)
        got = d[np.arange(len(d)), cell[s:s + 64]]
        # fp32 direct distances decide: D + 1 roundings in each of the two compared
        assert (got <= d.min(1) * (1 + 2 * (X.shape[1] + 1) * 2.0 ** -24)).all()


@pytest.mark.parametrize("nt", [1, 128, 129, 255, 256, 257, 640])
@pytest.mark.parametrize("D,k", [(32, 15), (64, 128), (96, 129), (128, 3 * 128), (128, 4 * 128 + 1), (32, 5 * 128 - 17), (96, 40 * 128)])
def test_strips_and_tiles(nt, D, k):
    rng = np.random.default_rng(nt + k)
    C = rng.normal(size=(k, D)).astype(np.float32)
    X = (C[rng.integers(0, k, nt)] + rng.normal(scale=0.4, size=(nt, D))).astype(np.float32)
    check(X, C, assign(X, C))


@pytest.mark.parametrize("D", [32, 128])
def test_rows_far_below_the_columns(D):
    """2^80 and more between the scales of the rows and of the columns, in one of a strip's two blocks."""
    rng = np.random.default_rng(D)
    k, nt = 400, 300
    C = rng.normal(size=(k // 2, D)) * 1e12 * (1 + np.arange(k // 2)[:, None] / k)
    C = np.concatenate([C, -C])  # the mean is zero: the rows are not shifted by it
    C[k - 1] = -C[k // 2 - 1] * 0.25
    X = rng.normal(size=(nt, D)) * 1e-20
    X[140:] = C[rng.integers(0, k, nt - 140)] * 1.01
    X, C = X.astype(np.float32), C.astype(np.float32)
    check(X, C, assign(X, C))


@pytest.mark.parametrize("D,k", [(64, 300), (128, 1000)])
def test_columns_that_do_not_count(D, k):
    """Centroids whose squared norm overflows (a pair that leaves the mean alone) are nobody's nearest."""
    rng = np.random.default_rng(1)
    nt = 200
    C = rng.normal(size=(k, D)).astype(np.float32)
    X = (C[rng.integers(0, k, nt)] + rng.normal(scale=0.4, size=(nt, D))).astype(np.float32)
    C[5, 7], C[k - 1, 7] = 1e25, -1e25
    cell = assign(X, C)
    assert not np.isin(cell, [5, k - 1]).any()
    check(X, C, cell)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("v", [1e20, 1e24, 1e37])
def test_columns_that_do_not_count_cost_nothing(D, v):
    """The same pair in a column block of its own: the other columns' shortlists stay short."""
    import paper_1901_00275_amd as vlq

    g = torch.Generator(device=DEV)
    g.manual_seed(2)
    k, nt = 64 * 128 + 2, 20_000
    C = torch.randn(k, D, generator=g, device=DEV)
    X = C[torch.randint(0, k - 2, (nt,), generator=g, device=DEV)] + 0.5 * torch.randn(nt, D, generator=g, device=DEV)
    cell = torch.empty(nt, dtype=torch.int32, device=DEV)

    def time_of():
        best = np.inf
        for _ in range(4):
            s, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            s.record()
            vlq.vlq_kmeans(X, nt, D, k, 0, C, cell, None)
            e.record()
            e.synchronize()
            best = min(best, s.elapsed_time(e))
        return best

    plain, want = time_of(), cell.clone()
    near = want < k - 2  # (vectors that were nearest to one of the pair go elsewhere)
    C[k - 2, 7], C[k - 1, 7] = v, -v
    assert time_of() < 2 * plain
    assert torch.equal(cell[near], want[near]) and (cell < k - 2).all()
