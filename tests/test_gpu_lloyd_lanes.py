"""Lloyd iterations of small codebooks of few dimensions (Sec. 2.1): the one-pass kernel against fp64."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


# nt around the lanes of a workgroup, more than one round of the grid; k around the batches of centroids, the largest
# whose sums fit the workgroup's LDS (and one more: the general path); off: vectors that are not 16-byte aligned
@pytest.mark.parametrize("nt,D,k,off", [
    (1, 16, 1, 0), (511, 16, 7, 0), (513, 12, 33, 1), (300_001, 16, 256, 0), (5_000, 16, 481, 0), (5_000, 16, 482, 0),
    (4_097, 6, 255, 1), (9_000, 4, 1_638, 0), (9_000, 8, 257, 3),
    # both sides of the choice between the one pass and the contraction
    (32_768, 16, 305, 0), (32_769, 16, 305, 0), (700, 16, 304, 0), (700, 12, 360, 0), (700, 12, 361, 0), (900, 8, 880, 0), (900, 6, 881, 0),
    (40_000, 16, 481, 0), (33_000, 8, 910, 0),
])
def test_one_pass_iteration(nt, D, k, off):
    import paper_1901_00275_amd as vlq

    rng = np.random.default_rng(nt + D + k)
    X = rng.normal(scale=20.0, size=(nt, D)).astype(np.float32)
    C = X[rng.integers(0, nt, k)] + rng.normal(scale=5.0, size=(k, D)).astype(np.float32)
    if k > 4:
        C[k // 2] = C[1]  # coinciding centroids: the smaller index
        C[3] = 1e4        # no members
    buf = torch.zeros(nt * D + off, device=DEV)
    Xd = buf[off:].view(nt, D)
    Xd.copy_(torch.as_tensor(X))
    Cd = torch.as_tensor(C).to(DEV)
    a = torch.empty(nt, dtype=torch.int32, device=DEV)
    n = torch.empty(k, dtype=torch.int32, device=DEV)
    vlq.vlq_kmeans(Xd, nt, D, k, 0, Cd, a, n)
    assert np.array_equal(Cd.cpu().numpy(), C)
    cell = a.cpu().numpy()
    X64, C64 = X.astype(np.float64), C.astype(np.float64)
    d = np.empty(nt)
    best = np.empty(nt)
    first = np.empty(nt, dtype=np.int64)
    for s in range(0, nt, 4096):
        dd = ((X64[s:s + 4096, None, :] - C64[None]) ** 2).sum(2)
        first[s:s + 4096] = dd.argmin(1)
        best[s:s + 4096] = dd.min(1)
        d[s:s + 4096] = dd[np.arange(len(dd)), cell[s:s + 4096]]
    # D + 1 roundings of fp32 in every distance, two distances compared
    assert (d <= best * (1 + 2 * (D + 1) * 2.0 ** -24)).all()
    assert np.array_equal(cell[d == best], first[d == best])
    assert np.array_equal(n.cpu().numpy(), np.bincount(cell, minlength=k))
    # the iteration moves every centroid to the mean of these members; fixed-point sums, one rounding to fp32
    vlq.vlq_kmeans(Xd, nt, D, k, 1, Cd, None, None)
    want = C64.copy()
    for c in np.unique(cell):
        want[c] = X64[cell == c].mean(0)
    assert (np.abs(Cd.cpu().numpy() - want) <= 2.0 ** -24 * np.abs(want) * (1 + 1e-6) + 1e-9).all()


def test_few_vectors_and_many_centroids_take_no_longer():
    """A lane's walk over 630 centroids outlasts the contraction when only a few workgroups have vectors (1.45 times)."""
    import paper_1901_00275_amd as vlq

    def ms(nt, D, k):
        X, C0 = torch.randn(nt, D, device=DEV), torch.randn(k, D, device=DEV)
        best = float("inf")
        for _ in range(5):
            C = C0.clone()
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            vlq.vlq_kmeans(X, nt, D, k, 20, C, None, None)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1))
        return best

    # D = 13 has no one-pass form: the same contraction, one dimension more
    assert ms(3_000, 12, 630) < 1.35 * ms(3_000, 13, 630)
