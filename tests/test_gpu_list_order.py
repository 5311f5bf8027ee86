"""Lists of an index with few points a list: those of up to 16 points, a few longer ones and a very long one among them, in
order of id with their own codes and lambda bytes; and the same where lists are long on average."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [5, 8, 16])
@pytest.mark.parametrize("k,n,N,long", [(7, 3, 40, 0), (100, 8, 3000, 17), (100, 8, 9000, 1500), (33, 4, 2000, 0), (5, 4, 5000, 300)])
def test_lists_are_in_order_of_id(m, k, n, N, long):
    import paper_1901_00275_amd as vlq

    rng = np.random.default_rng(k + N + m)
    D = 4 * m
    C = torch.tensor(rng.normal(size=(k, D)), dtype=torch.float32, device=DEV)
    P = torch.tensor(rng.normal(size=(m, 256, 4)), dtype=torch.float32, device=DEV)
    cell, edge = rng.integers(0, k, N), rng.integers(0, n, N)
    if long:
        cell[:long], edge[:long] = 1, 2
    ids = rng.permutation(5 * N)[:N]
    ids[: N // 10] = ids[N // 10 - 1]  # some ids repeat
    lam, codes = rng.integers(0, 256, N), rng.integers(0, 256, (N, m))
    t = lambda a, dt: torch.tensor(a).to(dt).to(DEV)
    idx = vlq.vlq_build_index(vlq.vlq_params_t(D, k, n, m, 0.0, 0.0), C, P)
    try:
        vlq.vlq_index_add_encoded(idx, t(cell, torch.int32), t(edge, torch.int32), t(lam, torch.uint8), t(codes, torch.uint8),
                                  t(ids, torch.int32), N)
        vlq.vlq_index_finalize(idx)
        off = torch.empty(k * n + 1, dtype=torch.int64, device=DEV)
        oid, olam = torch.empty(N, dtype=torch.int32, device=DEV), torch.empty(N, dtype=torch.uint8, device=DEV)
        ocode = torch.empty(N, m, dtype=torch.uint8, device=DEV)
        vlq.vlq_index_get_lists(idx, off, oid, ocode, olam)
        torch.cuda.synchronize()
    finally:
        vlq.vlq_index_free(idx)
    label = cell * n + edge
    assert np.array_equal(off.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(label, minlength=k * n))]))
    oid, olam, ocode = oid.cpu().numpy(), olam.cpu().numpy(), ocode.cpu().numpy()
    order = np.lexsort((ids, label))
    assert np.array_equal(oid, ids[order])
    # points of one list and id in any order: compare them as sorted records
    rec = lambda i, a, c: np.sort(np.array([f"{x:9d} {y:3d} {bytes(z).hex()}" for x, y, z in zip(i, a, c)]))
    off = off.cpu().numpy()
    for l in np.unique(label):
        s, e = off[l], off[l + 1]
        mine = np.flatnonzero(label == l)
        assert np.array_equal(rec(oid[s:e], olam[s:e], ocode[s:e]), rec(ids[mine], lam[mine].astype(np.uint8), codes[mine].astype(np.uint8)))
