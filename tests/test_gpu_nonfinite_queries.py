"""Queries that are not finite, or whose squares overflow, among ordinary ones: cells and sub-regions stay in range, the
ordinary queries keep their rows."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV, dev, make_index, vlq  # noqa: F401  (vlq: fixture)
from test_gpu_scan_wide import add
from util import Problem

pytestmark = pytest.mark.gpu


# k below one and several rounds of the register-resident selection's threads (its last round reaches past the end)
@pytest.mark.parametrize("D", [60, 32])
@pytest.mark.parametrize("k", [16, 1000, 1025, 4100, 17_000])
def test_indices_stay_in_range(vlq, D, k):  # noqa: F811
    rng = np.random.default_rng(k + D)
    n, m, nq, w1, w2, K = 4, D // 4, 20, 8, 20, 10
    C = rng.normal(size=(k, D)).astype(np.float32)
    pr = Problem("other", None, (C[rng.integers(0, k, nq)] + 0.3 * rng.normal(size=(nq, D))).astype(np.float32), C,
                 (0.3 * rng.normal(size=(m, 256, 4))).astype(np.float32), n)
    idx = make_index(vlq, pr)
    try:
        add(vlq, idx, pr, 20_000, k)

        def search(Y, fp32):
            vlq.vlq_index_set_option(idx, vlq.VLQ_OPT_COARSE_FP32, fp32)
            d, i = torch.empty(nq, K, device=DEV), torch.empty(nq, K, dtype=torch.int32, device=DEV)
            cells, cd = torch.empty(nq, w1, dtype=torch.int32, device=DEV), torch.empty(nq, w1, device=DEV)
            sub, ss = torch.empty(nq, w2, dtype=torch.int32, device=DEV), torch.empty(nq, w2, device=DEV)
            vlq.vlq_search_debug(idx, dev(Y), nq, w1, w2, K, d, i, cells, cd, sub, ss)
            return [t.cpu().numpy() for t in (d, i, cells, sub)]

        Y = pr.Y.copy()
        Y[3, 1], Y[7, 0], Y[11], Y[12, 5] = np.inf, np.nan, 1e25, -np.inf
        fine = np.isfinite(Y).all(1)
        fine[11] = False
        for fp32 in (1, 0):
            want, got = search(pr.Y, fp32), search(Y, fp32)
            for w, g in zip(want, got):
                assert np.array_equal(w[fine], g[fine])
            assert ((got[2] >= -1) & (got[2] < k)).all() and ((got[3] >= -1) & (got[3] < k * n)).all()
            assert ((got[1] >= -1) & (got[1] < 20_000)).all()
    finally:
        vlq.vlq_index_free(idx)


@pytest.mark.parametrize("D,k,nq", [(128, 4096, 1), (128, 4100, 5), (32, 16_384, 9), (60, 65_536, 2), (64, 5000, 64)])
def test_every_nan_takes_the_same_cells(vlq, D, k, nq):  # noqa: F811
    """A query of NaNs in a small batch, of the usual pattern and of the largest there is: the first cells, whatever the pattern."""
    rng = np.random.default_rng(k + D)
    n, m, w1, w2, K = 4, D // 4, 8, 20, 10
    C = rng.normal(size=(k, D)).astype(np.float32)
    pr = Problem("other", None, C[:nq].copy(), C, (0.3 * rng.normal(size=(m, 256, 4))).astype(np.float32), n)
    idx = make_index(vlq, pr)
    try:
        add(vlq, idx, pr, 20_000, k)

        def cells_of(Y):
            d, i = torch.empty(nq, K, device=DEV), torch.empty(nq, K, dtype=torch.int32, device=DEV)
            cells, cd = torch.empty(nq, w1, dtype=torch.int32, device=DEV), torch.empty(nq, w1, device=DEV)
            sub, ss = torch.empty(nq, w2, dtype=torch.int32, device=DEV), torch.empty(nq, w2, device=DEV)
            vlq.vlq_search_debug(idx, dev(Y), nq, w1, w2, K, d, i, cells, cd, sub, ss)
            return cells.cpu().numpy()

        usual, ones = pr.Y.copy(), pr.Y.copy()
        usual[nq // 2] = np.nan
        ones[nq // 2] = np.array(0x7FFFFFFF, np.uint32).view(np.float32)
        got = cells_of(usual)
        assert np.array_equal(got[nq // 2], np.arange(w1)) and np.array_equal(got, cells_of(ones))
    finally:
        vlq.vlq_index_free(idx)
