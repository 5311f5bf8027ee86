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
    def lists(rng):
        cell, edge = rng.integers(0, k, N), rng.integers(0, n, N)
        if long:
            cell[:long], edge[:long] = 1, 2
        return cell, edge

    check(m, k, n, N, lists, np.random.default_rng(k + N + m))


@pytest.mark.parametrize("m", [1, 6, 8, 64])
@pytest.mark.parametrize("k", [500, 300, 120])  # 4.3 points a list, 7.2 and 18
@pytest.mark.parametrize("sizes", [[2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 66, 127, 300, 1023, 1024, 1025, 1500], [64] * 100, [65] * 100, [17] * 64 + [64] * 64])
def test_crowded_cells(m, k, sizes):
    """Lists of every size class next to each other, among many of few points or none."""
    n, N = 8, 17_000

    def lists(rng):
        label = np.repeat(np.arange(len(sizes)) + 5, sizes)
        label = np.concatenate([label, rng.integers(len(sizes) + 9, k * n, N - len(label))])
        rng.shuffle(label)
        return label // n, label % n

    check(m, k, n, N, lists, np.random.default_rng(m + k + len(sizes)))


def check(m, k, n, N, lists, rng):
    import paper_1901_00275_amd as vlq

    D = 4 * m
    C = torch.tensor(rng.normal(size=(k, D)), dtype=torch.float32, device=DEV)
    P = torch.tensor(rng.normal(size=(m, 256, 4)), dtype=torch.float32, device=DEV)
    cell, edge = lists(rng)
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


def finalise_time(k, n, cell, edge, m=8, D=32):
    """Milliseconds of vlq_index_finalize over points in these lists, in random order."""
    import time

    import paper_1901_00275_amd as vlq

    N = len(cell)
    g = torch.Generator(device=DEV)
    g.manual_seed(k)
    C, P = torch.randn(k, D, generator=g, device=DEV), torch.randn(m, 256, D // m, generator=g, device=DEV)
    idx = vlq.vlq_build_index(vlq.vlq_params_t(D, k, n, m, 0.0, 0.0), C, P)
    try:
        lam = torch.full((N,), 100, dtype=torch.uint8, device=DEV)
        codes = torch.randint(0, 256, (N, m), generator=g, device=DEV, dtype=torch.uint8)
        vlq.vlq_index_add_encoded(idx, cell, edge, lam, codes, None, N)
        best = np.inf
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            vlq.vlq_index_finalize(idx)
            best = min(best, time.perf_counter() - t)
    finally:
        vlq.vlq_index_free(idx)
    return best * 1e3


def test_crowded_cells_of_an_empty_index_are_no_slower():
    """Two million points in 40 cells: with 16 384 cells (few points a list on average) and with 1 000 (many)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    n, N = 64, 2_000_000
    cell = torch.randint(0, 40, (N,), generator=g, device=DEV, dtype=torch.int32)
    edge = torch.randint(0, n, (N,), generator=g, device=DEV, dtype=torch.int32)
    empty = finalise_time(16_384, n, cell[:1000], edge[:1000])
    assert finalise_time(16_384, n, cell, edge) < 1.5 * finalise_time(1000, n, cell, edge) + empty


def test_a_long_list_among_short_ones_is_no_slower():
    """Half of 600 000 points in one list, the others spread: with 16 384 cells and with 100."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    n, N = 32, 600_000
    cell = torch.randint(0, 100, (N,), generator=g, device=DEV, dtype=torch.int32)
    edge = torch.randint(0, n, (N,), generator=g, device=DEV, dtype=torch.int32)
    cell[::2], edge[::2] = 5, 3
    empty = finalise_time(16_384, n, cell[1:1000:2].contiguous(), edge[1:1000:2].contiguous())
    assert finalise_time(16_384, n, cell, edge) < 1.3 * finalise_time(100, n, cell, edge) + empty


def test_both_sides_of_the_line_between_short_and_long_lists():
    """2 048 cells of 8 edges filled unevenly, with 16 points a list on average and with one point more."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1)
    k, n = 2048, 8
    N = 16 * k * n
    cell = torch.rand(N + 1, generator=g, device=DEV).pow_(2).mul_(k).to(torch.int32).clamp_(max=k - 1)
    edge = torch.rand(N + 1, generator=g, device=DEV).pow_(1.3).mul_(n).to(torch.int32).clamp_(max=n - 1)
    assert finalise_time(k, n, cell[:N], edge[:N], 16, 96) < 1.2 * finalise_time(k, n, cell, edge, 16, 96)


@pytest.mark.parametrize("m,ds", [(8, 4), (16, 6), (8, 5)])
@pytest.mark.parametrize("k", [1200, 500, 60])  # 1.8 points a list, 4.3 and 36; more than 8 192 lists, fewer
def test_static_terms_of_every_list(m, ds, k):
    """Distances to points of lists of every size class, against fp64: short lists, long ones among them, long ones all."""
    import paper_1901_00275_amd as vlq

    sizes, n, N, D, K = [1, 2, 15, 16, 17, 63, 64, 65, 66, 128, 129, 700, 1025], 8, 17_000, m * ds, 100
    rng = np.random.default_rng(m + ds + k)
    label = np.repeat(np.arange(len(sizes)) + 5, sizes)
    label = np.concatenate([label, rng.integers(len(sizes) + 9, k * n, N - len(label))])
    lam, codes = rng.integers(0, 256, N), rng.integers(0, 256, (N, m))
    C, P = rng.normal(size=(k, D)).astype(np.float32), (0.3 * rng.normal(size=(m, 256, ds))).astype(np.float32)
    t = lambda a, dt: torch.tensor(a).to(dt).to(DEV)  # noqa: E731
    idx = vlq.vlq_build_index(vlq.vlq_params_t(D, k, n, m, 0.0, 0.0), t(C, torch.float32), t(P, torch.float32))
    try:
        S, E = torch.empty(k, n, dtype=torch.int32, device=DEV), torch.empty(k, n, device=DEV)
        vlq.vlq_index_get_graph(idx, S, E)
        S = S.cpu().numpy()
        lh = (lam * 0.75 / 255 - 0.25)[:, None]  # the default grid
        c, s = C[label // n].astype(np.float64), C[S[label // n, label % n]].astype(np.float64)
        X = c + lh * (s - c) + P[np.arange(m), codes].reshape(N, D)
        seen = np.concatenate([np.flatnonzero(label == 5 + i)[:70] for i in range(len(sizes))] + [rng.integers(0, N, 100)])
        Y = (X[seen] + 1e-2 * rng.normal(size=(len(seen), D))).astype(np.float32)
        nq = len(Y)
        vlq.vlq_index_add_encoded(idx, t(label // n, torch.int32), t(label % n, torch.int32), t(lam, torch.uint8), t(codes, torch.uint8), None, N)
        vlq.vlq_index_finalize(idx)
        dist, ids = torch.empty(nq, K, device=DEV), torch.empty(nq, K, dtype=torch.int32, device=DEV)
        vlq.vlq_search(idx, t(Y, torch.float32), nq, min(k, 64), min(k, 64) * n, K, dist, ids)
        torch.cuda.synchronize()
    finally:
        vlq.vlq_index_free(idx)
    dist, ids = dist.cpu().numpy(), ids.cpu().numpy()
    found = 0
    for q in range(nq):
        d = ((Y[q].astype(np.float64) - X[ids[q]]) ** 2).sum(1)
        # fp32 sums of terms of the size of ||y||^2 and ||x||^2 + ||s - c||^2, a hundred roundings at most
        assert (np.abs(dist[q] - d) < 100 * 2.0 ** -24 * 8 * ((Y[q] ** 2).sum() + (X[ids[q]] ** 2).sum(1) + 4 * D)).all()
        found += seen[q] in ids[q]
    assert found > 0.95 * nq
