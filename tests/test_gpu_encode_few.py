"""Small batches (four vectors per workgroup) encode to the rows of the large batch (64 per workgroup) bit for bit."""
import numpy as np
import pytest

from test_gpu_parity import gpu_encode, make_index, vlq  # noqa: F401  (vlq: fixture)
from util import problem

pytestmark = pytest.mark.gpu


# sub-spaces of 4, 6, 8, 12 and 16 dimensions, D below and above 64, n not a multiple of the 16 rows of a round
@pytest.mark.parametrize("D,m,n", [(32, 8, 7), (96, 16, 32), (128, 16, 33), (96, 8, 16), (128, 8, 5), (60, 10, 1)])
def test_small_batches_encode_like_large_ones(vlq, D, m, n):  # noqa: F811
    pr = problem(N=9000, k=70, n=n, m=m, G=16, nq=2, D=D, iters=1)
    idx = make_index(vlq, pr)
    try:
        X = np.concatenate([pr.X, pr.X[:1] * np.nan])  # a vector without a nearest centroid stays in range
        want = gpu_encode(vlq, idx, X, m)
        for at, nb in ((0, 1), (0, 3), (4, 5), (11, 100), (8800, 201), (0, 8192)):
            got = gpu_encode(vlq, idx, X[at:at + nb], m)
            for g, w in zip(got, want):
                assert np.array_equal(g, w[at:at + nb]), (at, nb)
    finally:
        vlq.vlq_index_free(idx)
