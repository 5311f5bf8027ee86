"""The cut of the sub-regions kept in registers against the general kernel (which vlq_search_debug takes): numbers of edges
that are multiples of four and others, 4, 8 and 16 keys a thread, all and few sub-regions wanted, equal scores at the cut."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w1,n,w2", [(4, 4, 16), (8, 6, 11), (16, 8, 1), (31, 8, 100), (64, 16, 1024), (33, 32, 200), (64, 32, 2048),
                                     (21, 48, 333), (64, 64, 1024), (63, 64, 2000), (40, 50, 499)])
@pytest.mark.parametrize("same", [False, True])
def test_same_lists_as_the_general_kernel(w1, n, w2, same):
    import paper_1901_00275_amd as vlq

    rng = np.random.default_rng(w1 * n + w2)
    k, D, m, nq, K, N = 200, 32, 8, 70, 50, 20_000
    C = rng.normal(size=(k, D))
    if same:  # every centroid three times: edges of length zero, equal scores
        C = np.repeat(C[: k // 3 + 1], 3, 0)[:k]
    C = torch.tensor(C, dtype=torch.float32, device=DEV)
    P = torch.tensor(rng.normal(size=(m, 256, D // m)) * 0.3, dtype=torch.float32, device=DEV)
    Y = torch.tensor(rng.normal(size=(nq, D)), dtype=torch.float32, device=DEV)
    idx = vlq.vlq_build_index(vlq.vlq_params_t(D, k, n, m, 0.0, 0.0), C, P)
    try:
        g = torch.Generator(device=DEV)
        g.manual_seed(1)
        cell = torch.randint(0, k, (N,), generator=g, device=DEV, dtype=torch.int32)
        edge = torch.randint(0, n, (N,), generator=g, device=DEV, dtype=torch.int32)
        lam = torch.randint(0, 256, (N,), generator=g, device=DEV, dtype=torch.int32).to(torch.uint8)
        codes = torch.randint(0, 256, (N, m), generator=g, device=DEV, dtype=torch.int32).to(torch.uint8)
        vlq.vlq_index_add_encoded(idx, cell, edge, lam, codes, None, N)
        vlq.vlq_index_finalize(idx)
        got = torch.empty(nq, K, device=DEV), torch.empty(nq, K, dtype=torch.int32, device=DEV)
        ref = torch.empty(nq, K, device=DEV), torch.empty(nq, K, dtype=torch.int32, device=DEV)
        vlq.vlq_search(idx, Y, nq, w1, w2, K, *got)
        cells, cd = torch.empty(nq, w1, dtype=torch.int32, device=DEV), torch.empty(nq, w1, device=DEV)
        sub, ss = torch.empty(nq, w2, dtype=torch.int32, device=DEV), torch.empty(nq, w2, device=DEV)
        vlq.vlq_search_debug(idx, Y, nq, w1, w2, K, *ref, cells, cd, sub, ss)
        torch.cuda.synchronize()
    finally:
        vlq.vlq_index_free(idx)
    # the same lists are scanned by the same kernel (in another order: equal distances at the K-th place may differ)
    assert torch.equal(got[0], ref[0])
    inside = ref[0] < ref[0][:, -1:]
    assert torch.equal(got[1][inside], ref[1][inside])
