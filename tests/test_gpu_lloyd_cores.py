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
