"""The streaming scan's K-selection on whole-number data, where every distance is exact and most of them are shared: the K
smallest by (distance, place in the lists), returned by (distance, id).  Few points and many, one result to 128, short lists
(several to a chunk) and long ones."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [8, 16])
@pytest.mark.parametrize("N,spread,K", [(0, 1, 5), (1, 1, 3), (90, 1, 128), (700, 1, 100), (700, 9, 127), (1500, 0, 128), (5000, 9, 1),
                                        (5000, 2, 8), (5000, 40, 9), (900, 300, 128), (1000, 0, 120),
                                        (1000, 40, 128), (30_000, 1, 128), (30_000, 300, 100), (30_000, 0, 10)])
def test_ties_and_order(m, N, spread, K):
    import paper_1901_00275_amd as vlq

    rng = np.random.default_rng(N + spread + K)
    k, n, D, nq = 8, 4, 4 * m, 1030  # (so many queries that none is split)
    C = rng.integers(-20, 21, (k // 2, D))
    C = torch.tensor(np.concatenate([C, -C]), dtype=torch.float32)  # the mean is zero
    P = torch.tensor(rng.integers(-spread, spread + 1, (m, 256, 4)), dtype=torch.float32)
    Y = torch.tensor(rng.integers(-30, 31, (nq, D)), dtype=torch.float32)
    Y[5] = Y[4]
    idx = vlq.vlq_build_index(vlq.vlq_params_t(D, k, n, m, 0.0, 0.0), C.to(DEV), P.to(DEV))
    try:
        if N:
            cell, edge = rng.integers(0, k, N), rng.integers(0, n, N)
            cell[: N // 3] = 2  # a long list
            edge[: N // 3] = 1
            codes = torch.tensor(rng.integers(0, 256, (N, m)), dtype=torch.uint8)
            ids = torch.tensor(rng.permutation(N).astype(np.int32) // 2)  # every id twice
            vlq.vlq_index_add_encoded(idx, torch.tensor(cell, dtype=torch.int32).to(DEV), torch.tensor(edge, dtype=torch.int32).to(DEV),
                                      torch.full((N,), 85, dtype=torch.uint8).to(DEV), codes.to(DEV), ids.to(DEV), N)
            vlq.vlq_index_finalize(idx)
        off = torch.empty(k * n + 1, dtype=torch.int64, device=DEV)
        lids, lam = torch.empty(max(N, 1), dtype=torch.int32, device=DEV), torch.empty(max(N, 1), dtype=torch.uint8, device=DEV)
        lcodes = torch.empty(max(N, 1), m, dtype=torch.uint8, device=DEV)
        if N:
            vlq.vlq_index_get_lists(idx, off, lids, lcodes, lam)
        dist, out = torch.empty(nq, K, device=DEV), torch.empty(nq, K, dtype=torch.int32, device=DEV)
        vlq.vlq_search(idx, Y.to(DEV), nq, k, k * n, K, dist, out)
        torch.cuda.synchronize()
    finally:
        vlq.vlq_index_free(idx)
    dist, out = dist.cpu().numpy(), out.cpu().numpy()
    take = min(K, N)
    assert (out[:, take:] == -1).all() and np.isinf(dist[:, take:]).all()
    if not N:
        return
    off, lids, lcodes = off.cpu().numpy(), lids.cpu().numpy(), lcodes.cpu().numpy()
    where = np.repeat(np.arange(k * n), np.diff(off)) // n
    X = C.numpy()[where] + P.numpy()[np.arange(m), lcodes].reshape(N, D)  # lambda is zero everywhere
    for q in range(0, nq, 37 if N > 10_000 else 11):
        d = ((Y.numpy()[q] - X) ** 2).sum(1, dtype=np.float64)
        kept = np.lexsort((np.arange(N), d))[:take]
        kept = kept[np.lexsort((lids[kept], d[kept]))]
        assert np.array_equal(dist[q, :take], d[kept]), q
        assert np.array_equal(out[q, :take], lids[kept]), q
    assert np.array_equal(dist[4], dist[5]) and np.array_equal(out[4], out[5])


@pytest.mark.parametrize("nq", [1, 17, 300])
def test_split_queries_return_the_same_distances(nq):
    """Queries split over workgroups: the same distances, each id at the distance it has."""
    import paper_1901_00275_amd as vlq

    rng = np.random.default_rng(nq)
    m, k, n, N, K = 8, 16, 8, 4000, 100
    D = 4 * m
    C = rng.integers(-20, 21, (k // 2, D))
    C = torch.tensor(np.concatenate([C, -C]), dtype=torch.float32)
    P = torch.tensor(rng.integers(-2, 3, (m, 256, 4)), dtype=torch.float32)
    Y = torch.tensor(rng.integers(-30, 31, (nq, D)), dtype=torch.float32)
    cell, edge = rng.integers(0, k, N), rng.integers(0, n, N)
    codes = rng.integers(0, 256, (N, m))
    idx = vlq.vlq_build_index(vlq.vlq_params_t(D, k, n, m, 0.0, 0.0), C.to(DEV), P.to(DEV))
    try:
        vlq.vlq_index_add_encoded(idx, torch.tensor(cell, dtype=torch.int32).to(DEV), torch.tensor(edge, dtype=torch.int32).to(DEV),
                                  torch.full((N,), 85, dtype=torch.uint8).to(DEV), torch.tensor(codes, dtype=torch.uint8).to(DEV), None, N)
        vlq.vlq_index_finalize(idx)
        dist, out = torch.empty(nq, K, device=DEV), torch.empty(nq, K, dtype=torch.int32, device=DEV)
        vlq.vlq_search(idx, Y.to(DEV), nq, k, k * n, K, dist, out)
        torch.cuda.synchronize()
    finally:
        vlq.vlq_index_free(idx)
    dist, out = dist.cpu().numpy(), out.cpu().numpy()
    X = C.numpy()[cell] + P.numpy()[np.arange(m), codes].reshape(N, D)
    for q in range(nq):
        d = ((Y.numpy()[q] - X) ** 2).sum(1, dtype=np.float64)
        assert np.array_equal(dist[q], np.sort(d)[:K])
        assert np.array_equal(d[out[q]], dist[q]) and len(set(out[q])) == K
        same = np.diff(dist[q]) == 0
        assert (np.diff(out[q])[same] > 0).all()
