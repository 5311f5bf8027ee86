"""The scan for K > 128 and for code lengths other than 8 and 16 against the 2m-lookup scan: many turns of the
workgroup (the candidate buffer is cut several times), one point per list, one long list, K at its limits, split
queries, and points that coincide in distance and id (more of them than the candidate buffer holds)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import DEV, dev, gpu_search, make_index, vlq  # noqa: F401  (vlq: fixture)
from util import Problem, problem

pytestmark = pytest.mark.gpu


def both_scans(vlq, idx, Y, w1, w2, K):  # noqa: F811
    out = []
    for generic in (1, 0):
        vlq.vlq_index_set_option(idx, vlq.VLQ_OPT_SCAN_GENERIC, generic)
        out.append(gpu_search(vlq, idx, Y, w1, w2, K)[:2])
    return out


def add(vlq, idx, pr, N, cells, ids=None, same=False, seed=0):  # noqa: F811
    rng = np.random.default_rng(seed)
    cell = rng.integers(0, cells, N).astype(np.int32)
    edge = rng.integers(0, pr.n, N).astype(np.int32)
    lam = rng.integers(60, 256, N).astype(np.uint8)
    codes = rng.integers(0, 256, (N, pr.m)).astype(np.uint8)
    if same:
        cell[:], edge[:], lam[:], codes[:] = 0, 0, 100, 7
    vlq.vlq_index_add_encoded(idx, dev(cell), dev(edge), dev(lam), dev(codes), None if ids is None else dev(ids), N)
    vlq.vlq_index_finalize(idx)


@pytest.mark.parametrize(
    "m,D,K,N,cells,nq",
    [(8, 32, 129, 60_000, 32, 40), (8, 128, 1000, 60_000, 32, 40), (16, 96, 1024, 60_000, 32, 3), (10, 60, 1, 20_000, 32, 33),
     (10, 60, 1000, 50_000, 32, 1500), (20, 100, 128, 30_000, 32, 20), (5, 35, 200, 30_000, 32, 20), (1, 3, 300, 5_000, 32, 20),
     (32, 128, 100, 30_000, 32, 20), (64, 128, 1024, 30_000, 32, 20), (8, 32, 1000, 40, 32, 20), (8, 32, 500, 30_000, 1, 1)])
def test_wide_scan_equals_generic(vlq, m, D, K, N, cells, nq):  # noqa: F811
    pr = problem(N=2000, k=32, n=4, m=m, G=16, nq=nq, D=D, iters=1)
    idx = make_index(vlq, pr)
    try:
        add(vlq, idx, pr, N, cells)
        (dg, ig), (dw, iw) = both_scans(vlq, idx, pr.Y, 16, 60, K)
        # the result's distances are the 2m-lookup scan's own, bit for bit
        assert np.array_equal(dg, dw) and np.array_equal(ig, iw)
    finally:
        vlq.vlq_index_free(idx)


@pytest.mark.parametrize("same_ids", [False, True])
@pytest.mark.parametrize("K", [129, 1000])
def test_coinciding_points(vlq, K, same_ids):  # noqa: F811
    """30 000 copies of one point: the smallest ids stay; with one id for all of them, K times that id."""
    pr = problem(N=2000, k=32, n=4, m=8, G=16, nq=40, D=32, iters=1)
    idx = make_index(vlq, pr)
    try:
        N = 30_000
        ids = np.full(N, 5, np.int32) if same_ids else np.random.default_rng(1).permutation(N).astype(np.int32)
        add(vlq, idx, pr, N, 1, ids=ids, same=True)
        d, i = (torch.empty(40, K, device=DEV), torch.empty(40, K, dtype=torch.int32, device=DEV))
        vlq.vlq_search(idx, dev(pr.Y), 40, 32, 128, K, d, i)
        torch.cuda.synchronize()
        d, i = d.cpu().numpy(), i.cpu().numpy()
        assert (d == d[:, :1]).all() and np.isfinite(d).all()
        assert (i == (5 if same_ids else np.arange(K))).all()
    finally:
        vlq.vlq_index_free(idx)


def clusters(k, n, m, D, spread, nq, seed=0):
    """Tight clusters far from the centroids' mean: distances are small against what the scan's table is made of."""
    rng = np.random.default_rng(seed)
    C = np.repeat(rng.normal(size=((k + 31) // 32, D)), 32, 0)[:k] + spread * rng.normal(size=(k, D))
    P = spread * rng.normal(size=(m, 256, D // m))
    Y = C[rng.integers(0, k, nq)] + spread * rng.normal(size=(nq, D))
    return Problem("other", None, *(v.astype(np.float32) for v in (Y, C, P)), n)


# (64, 1 024, 2 048 lists and a workgroup per query: the largest LDS image of the kernel)
@pytest.mark.parametrize("m,D,k,n,K,N,nq,w1,w2", [
    (64, 1024, 64, 32, 1024, 150_000, 1024, 64, 2048), (64, 1024, 64, 32, 1024, 150_000, 2, 64, 2048), (8, 128, 64, 8, 1000, 400_000, 300, 16, 100)])
@pytest.mark.parametrize("spread", [1.0, 0.02, 1e-3])
def test_clusters(vlq, m, D, k, n, K, N, nq, w1, w2, spread):  # noqa: F811
    pr = clusters(k, n, m, D, spread, nq)
    idx = make_index(vlq, pr)
    try:
        add(vlq, idx, pr, N, k)
        (dg, ig), (dw, iw) = both_scans(vlq, idx, pr.Y, w1, w2, K)
        assert np.array_equal(dg, dw) and np.array_equal(ig, iw)
    finally:
        vlq.vlq_index_free(idx)


def scan_times(vlq, idx, Y, w1, w2, K):  # noqa: F811
    """milliseconds of the 2m-lookup scan and of this one"""
    Yd, out = dev(Y), []
    d, i = torch.empty(len(Y), K, device=DEV), torch.empty(len(Y), K, dtype=torch.int32, device=DEV)
    for generic in (1, 0):
        vlq.vlq_index_set_option(idx, vlq.VLQ_OPT_SCAN_GENERIC, generic)
        best = float("inf")
        for _ in range(4):
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            vlq.vlq_search(idx, Yd, len(Y), w1, w2, K, d, i)
            t1.record()
            t1.synchronize()
            best = min(best, t0.elapsed_time(t1))
        out.append(best)
    return out


def test_clusters_are_not_slower(vlq):  # noqa: F811
    """Tight clusters in long lists: too wide a bound kept more points than the buffer holds, and the scan started over."""
    pr = clusters(64, 8, 8, 128, 0.01, 256)
    idx = make_index(vlq, pr)
    try:
        add(vlq, idx, pr, 4_000_000, 64)
        generic, wide = scan_times(vlq, idx, pr.Y, 8, 16, 1000)
        assert wide < generic
    finally:
        vlq.vlq_index_free(idx)


def coinciding(vlq, pr, N, seed=0):  # noqa: F811
    """An index whose lists hold one point many times over, under ids in any order."""
    idx = make_index(vlq, pr)
    at = np.arange(N)
    vlq.vlq_index_add_encoded(idx, dev((at // pr.n % pr.k).astype(np.int32)), dev((at % pr.n).astype(np.int32)),
                              dev(np.full(N, 100, np.uint8)), dev(np.full((N, pr.m), 7, np.uint8)),
                              dev(np.random.default_rng(seed).permutation(N).astype(np.int32)), N)
    vlq.vlq_index_finalize(idx)
    return idx


# lists around the length from which workgroups hand over to the 2m-lookup scan (1 536 points, 256 for codes of more
# than 16 bytes), queries whose bound is not finite, split and unsplit
@pytest.mark.parametrize("m,D,length,nq", [(8, 64, 1535, 3), (8, 64, 1537, 3), (8, 64, 2500, 1100), (20, 60, 255, 20), (20, 60, 300, 20), (5, 35, 3000, 20)])
@pytest.mark.parametrize("nan_codeword", [False, True])
def test_long_lists_of_coinciding_points(vlq, m, D, length, nq, nan_codeword):  # noqa: F811
    pr = clusters(16, 4, m, D, 0.3, nq)
    pr.Y[nq // 2, 1] = np.inf
    pr.Y[nq // 3, 0] = np.nan
    if nan_codeword:
        pr.P[0, 7, 0] = np.nan
    idx = coinciding(vlq, pr, length * 64)
    try:
        out = []
        for generic in (1, 0):
            vlq.vlq_index_set_option(idx, vlq.VLQ_OPT_SCAN_GENERIC, generic)
            d, i = torch.empty(nq, 1000, device=DEV), torch.empty(nq, 1000, dtype=torch.int32, device=DEV)
            vlq.vlq_search(idx, dev(pr.Y), nq, 8, 20, 1000, d, i)
            out.append((d.cpu().numpy(), i.cpu().numpy()))
        (dg, ig), (dw, iw) = out
        assert np.array_equal(dg, dw, equal_nan=True) and np.array_equal(ig, iw)
    finally:
        vlq.vlq_index_free(idx)


def test_coinciding_points_in_long_lists_are_not_slower(vlq):  # noqa: F811
    """More points within the bound than the buffer holds: taken one by one they took 3.5 times the 2m-lookup scan."""
    pr = clusters(64, 8, 8, 128, 0.3, 256)
    idx = coinciding(vlq, pr, 64 * 8 * 16_000)
    try:
        generic, wide = scan_times(vlq, idx, pr.Y, 8, 16, 1000)
        assert wide < 1.8 * generic
    finally:
        vlq.vlq_index_free(idx)


# around the lines of the choice: one list a workgroup and several, few and many points in it, rows of a sub-space on 16
# bytes and not
@pytest.mark.parametrize("m,D,length,w2,K", [
    (20, 120, 190, 4, 1000), (20, 120, 1000, 4, 1000), (20, 120, 16_000, 4, 1000), (20, 120, 1000, 16, 1000), (20, 120, 1000, 4, 10),
    (64, 256, 1000, 4, 1000), (32, 128, 1000, 4, 1000), (32, 128, 4000, 4, 1000), (5, 35, 1000, 4, 500), (8, 128, 1000, 4, 1000)])
def test_many_results_from_few_lists(vlq, m, D, length, w2, K):  # noqa: F811
    """The second scoring of all K outweighs a list's tables: twice the time of the 2m-lookup scan, which it was."""
    pr = clusters(16, 4, m, D, 0.3, 256)
    idx = make_index(vlq, pr)
    try:
        add(vlq, idx, pr, length * 64, 16)
        (dg, ig), (dw, iw) = both_scans(vlq, idx, pr.Y, 4, w2, K)
        assert np.array_equal(dg, dw) and np.array_equal(ig, iw)
        generic, chosen = scan_times(vlq, idx, pr.Y, 4, w2, K)
        assert chosen < 1.5 * generic
    finally:
        vlq.vlq_index_free(idx)


def test_second_launch_in_a_captured_graph(vlq):  # noqa: F811
    """Both launches of the scan replay from a graph: queries with something left for the second one, and without, in turn."""
    pr = clusters(16, 4, 8, 64, 0.3, 6)
    idx = coinciding(vlq, pr, 64 * 1800)
    try:
        Y, K = dev(pr.Y), 1000
        d, i = torch.empty(6, K, device=DEV), torch.empty(6, K, dtype=torch.int32, device=DEV)
        vlq.vlq_search_noalloc(idx, Y, 6, 8, 20, K, d, i)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            vlq.vlq_search_noalloc(idx, Y, 6, 8, 20, K, d, i)
        rng = np.random.default_rng(2)
        for turn in range(4):
            q = pr.Y[rng.permutation(6)].copy()
            if turn % 2:
                q[turn] = 1e25
            Y.copy_(torch.as_tensor(q))
            want_d, want_i = torch.empty_like(d), torch.empty_like(i)
            vlq.vlq_search(idx, dev(q), 6, 8, 20, K, want_d, want_i)
            torch.cuda.synchronize()
            d.fill_(-1)
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(i, want_i) and np.array_equal(d.cpu().numpy(), want_d.cpu().numpy(), equal_nan=True)
    finally:
        vlq.vlq_index_free(idx)
