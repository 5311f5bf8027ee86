"""Queries split over workgroups and merged (sorted lists of up to 16 workgroups) give the rows of the unsplit scan bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import gpu_search, make_index, vlq  # noqa: F401  (vlq: fixture)
from test_gpu_scan_wide import add
from util import problem

pytestmark = pytest.mark.gpu


# K around a wave, a workgroup and the limit of the stream scan; more splits than results, fewer points than results;
# 16 lists of 16 and of 17 results (where every key has a thread, and where not)
@pytest.mark.parametrize("m,K,N,w2", [
    (8, 1, 40_000, 64), (8, 16, 40_000, 64), (8, 17, 40_000, 64), (8, 37, 40_000, 60), (16, 64, 40_000, 64), (16, 65, 40_000, 3), (8, 100, 40_000, 64), (8, 128, 40_000, 33),
    (8, 129, 40_000, 64), (8, 256, 900, 64), (16, 1000, 40_000, 64), (8, 100, 50, 64),
])
def test_split_rows_equal_unsplit_rows(vlq, m, K, N, w2):  # noqa: F811
    pr = problem(N=2000, k=32, n=4, m=m, G=16, nq=1100, D=32, iters=1)
    idx = make_index(vlq, pr)
    try:
        add(vlq, idx, pr, N, 32)
        d, i = gpu_search(vlq, idx, pr.Y, 16, w2, K)[:2]
        for nq in (1, 2, 16, 17, 61, 300, 600):
            ds, js = gpu_search(vlq, idx, pr.Y[:nq], 16, w2, K)[:2]
            assert np.array_equal(ds, d[:nq]) and np.array_equal(js, i[:nq]), nq
    finally:
        vlq.vlq_index_free(idx)
