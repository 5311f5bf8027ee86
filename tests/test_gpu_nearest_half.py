"""Nearest centroid through the fp16 product against fp64: edges of tiles, splits and row blocks, many centroids inside the
band (slots and whole splits are searched exactly), rows and centroids of very different sizes."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


def assign(X, C):
    import paper_1901_00275_amd as vlq

    a = torch.empty(len(X), dtype=torch.int32, device=DEV)
    vlq.vlq_kmeans(torch.as_tensor(X).to(DEV), len(X), X.shape[1], len(C), 0, torch.as_tensor(C).to(DEV), a, None)
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
