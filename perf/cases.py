"""The work that a user of the index has it do, as cases that can be timed and compared.

Four kinds, all through the functions of ``paper_1901_00275_amd``:

* ``search``  a batch of queries against a finalised index (Alg. 3): ``vlq_search``, and
              ``vlq_search_noalloc`` for the callers that may not allocate;
* ``encode``  cell, edge, lambda byte and codes of new vectors (Alg. 1 and 2);
* ``build``   an index from base vectors: graph, encoding, inverted lists;
* ``train``   Lloyd iterations for a codebook.

Vectors are Gaussian mixtures with the dimension and the value range of the two collections the
configurations are modelled on: "sift" D = 128, integers in [0, 255]; "deep" D = 96, unit norm; other
dimensions as "deep" without the normalisation.  Centroids are drawn around the mixture's means, codewords
with the spread of the residuals, so nothing is trained or encoded to prepare a case.  The stored points of a
searched index are drawn as (cell, edge, lambda byte, code): cells of uneven size, near edges and small lambdas more often,
uniform code bytes, as encoded descriptors have them; queries are vectors of the mixture.
"""
import torch

import paper_1901_00275_amd as vlq

DEV = "cuda"
ADD_CHUNK = 1 << 26  # stored points handed to the index at a time


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _search(name, kind, N, k, n, m, nq, w1, w2, K, D=None, noalloc=False, **more):
    D = D or (128 if kind == "sift" else 96)
    return dict(name=name, do="search", kind=kind, D=D, N=N, k=k, n=n, m=m, nq=nq, w1=w1, w2=w2, K=K,
                noalloc=noalloc, **more)


def listed():
    return [
        # one query of an interactive user: nothing but latency
        _search("search_1", "deep", 100_000_000, 65_536, 32, 16, nq=1, w1=64, w2=512, K=10),
        # a server that answers a few users at a time and must not allocate
        _search("search_17_noalloc", "sift", 10_000_000, 16_384, 32, 8, nq=17, w1=32, w2=256, K=100, noalloc=True),
        # a server that collects requests for a moment
        _search("search_256", "deep", 250_000_000, 16_384, 64, 16, nq=256, w1=64, w2=1_024, K=10),
        # the whole query set of a collection at once, short lists: the traversal weighs as much as the scan
        _search("search_10000_mid", "sift", 10_000_000, 16_384, 32, 8, nq=10_000, w1=32, w2=256, K=100),
        # the same, 16-byte codes, long lists
        _search("search_10000_deep", "deep", 250_000_000, 16_384, 64, 16, nq=10_000, w1=64, w2=1_024, K=100),
        # the headline: 10^9 points, 10 000 queries
        _search("search_10000_billion", "sift", 1_000_000_000, 65_536, 32, 8, nq=10_000, w1=64, w2=512, K=100),
        # many results per query, for a re-ranking stage of the caller's own; an odd batch
        _search("search_1501_top1000", "sift", 10_000_000, 16_384, 32, 8, nq=1_501, w1=64, w2=512, K=1_000),
        # points that arrive a hundred at a time
        dict(name="encode_100", do="encode", kind="deep", D=96, k=65_536, n=32, m=16, nb=100),
        # a bulk load, not a multiple of anything
        dict(name="encode_1000003", do="encode", kind="sift", D=128, k=65_536, n=32, m=8, nb=1_000_003),
        # a whole index from its vectors
        dict(name="build_2M", do="build", kind="sift", D=128, k=16_384, n=32, m=8, N=2_000_000),
        # training: the first-level codebook, and one sub-space of the product quantiser
        dict(name="train_cells", do="train", kind="deep", D=96, k=16_384, nt=500_000, iters=2),
        dict(name="train_codewords", do="train", kind="sift", D=16, k=256, nt=262_144, iters=10),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    """One more case of the same ranges."""
    do = rng.choices(["search", "encode", "build", "train"], [6, 2, 1, 1])[0]
    kind = rng.choice(["sift", "sift", "deep", "deep", "other"])
    if kind == "sift":
        D, m = 128, rng.choice([8, 8, 16])
    elif kind == "deep":
        D, m = 96, rng.choice([16, 16, 8])
    else:  # sizes off the two collections: fp32 contractions and the scan with 2m lookups among them
        m = rng.choice([8, 10, 16, 20])
        D = m * rng.choice([4, 5, 6, 8])
    n = rng.choice([8, 16, 32, 32, 48, 64])
    if do == "search":
        nq = _log(rng, 1, 10_000)
        k = _log(rng, 1_000, 65_536)
        w1 = _log(rng, 4, 64)
        w2 = max(1, int(rng.choice([0.25, 0.25, 0.4]) * w1 * n))
        # list lengths from a few points to several hundred
        N = min(k * n * _log(rng, 5, 480), 250_000_000)
        K = _log(rng, 1, 128) if rng.random() < 0.85 else _log(rng, 129, 1_000)
        while nq > 1 and nq * w2 * (N / (k * n)) > (1.2e9 if K <= 128 and m in (8, 16) else 1e8):
            nq //= 2
        noalloc = nq <= 64 and rng.random() < 0.3
        return _search("", kind, N, k, n, m, nq, w1, w2, K, D=D, noalloc=noalloc) | {"name": "search"}
    if do == "encode":
        k = _log(rng, 1_000, 65_536)
        return dict(name="encode", do=do, kind=kind, D=D, k=k, n=n, m=m, nb=_log(rng, 1, 1_000_003))
    if do == "build":
        k = _log(rng, 500, 16_384)
        return dict(name="build", do=do, kind=kind, D=D, k=k, n=n, m=m, N=_log(rng, 10_000, 2_000_000))
    if rng.random() < 0.5:
        return dict(name="train", do=do, kind=kind, D=D, k=_log(rng, 500, 16_384), nt=_log(rng, 50_000, 500_000), iters=2)
    return dict(name="train", do=do, kind=kind, D=rng.choice([4, 6, 8, 12, 16]), k=256, nt=_log(rng, 20_000, 262_144), iters=10)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class Mixture:
    """Seeded vectors, centroids and codewords on the GPU."""

    def __init__(self, kind, D, components, seed):
        self.kind, self.D = kind, D
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)
        if kind == "sift":
            self.means, self.sigma = self.rand(components, D) * 128.0, 20.0
        else:
            self.means, self.sigma = self.randn(components, D), 0.3

    def rand(self, *shape):
        return torch.rand(*shape, generator=self.g, device=DEV)

    def randn(self, *shape):
        return torch.randn(*shape, generator=self.g, device=DEV)

    def vectors(self, count, spread=1.0):
        comp = torch.randint(0, self.means.shape[0], (count,), generator=self.g, device=DEV)
        x = self.randn(count, self.D).mul_(self.sigma * spread).add_(self.means[comp])
        if self.kind == "sift":
            x.clamp_(0.0, 255.0)
            if spread == 1.0:
                x.round_()
        elif self.kind == "deep":
            x.div_(x.norm(dim=1, keepdim=True))
        return x.contiguous()

    def centroids(self, k):
        """Around the means, a few to a component, closer in than the points themselves."""
        return self.vectors(k, spread=0.6)

    def codewords(self, m):
        scale = self.sigma / (float(self.D) ** 0.5 if self.kind == "deep" else 1.0)
        return (self.randn(m, 256, self.D // m) * scale).contiguous()


class Index:
    """Owner of a library handle."""

    def __init__(self, case, C, P, X=None):
        prm = vlq.vlq_params_t(case["D"], case["k"], case["n"], case["m"], 0.0, 0.0)
        self.h = vlq.vlq_build_index(prm, C, P) if X is None else vlq.vlq_build_index(prm, C, P, X, X.shape[0])

    def close(self):
        if self.h is not None:
            vlq.vlq_index_free(self.h)
            self.h = None

    __del__ = close


def _stored_points(case, mix, idx):
    """Fills and finalises an index with case["N"] encoded points."""
    N, k, n, m = case["N"], case["k"], case["n"], case["m"]
    place = torch.randperm(k, generator=mix.g, device=DEV).to(torch.int32)
    vlq.vlq_index_reserve(idx.h, N)
    for at in range(0, N, ADD_CHUNK):
        cnt = min(ADD_CHUNK, N - at)
        cell = place[mix.rand(cnt).pow_(1.2).mul_(k).to(torch.int32).clamp_(max=k - 1)]
        edge = mix.rand(cnt).pow_(1.3).mul_(n).to(torch.int32).clamp_(max=n - 1)
        lam = mix.rand(cnt).pow_(1.5).mul_(170.0).add_(85.0).to(torch.uint8)
        words = (cnt * m + 7) // 8
        codes = torch.empty(words, dtype=torch.int64, device=DEV).random_(-(2**63), None, generator=mix.g)
        codes = codes.view(torch.uint8)[: cnt * m].view(cnt, m)
        vlq.vlq_index_add_encoded(idx.h, cell, edge, lam, codes, None, cnt)
    vlq.vlq_index_finalize(idx.h)


def prepare(case, seed):
    """Inputs and handles in the user's hands before the call."""
    do, k, D = case["do"], case["k"], case["D"]
    if do == "train":
        # cells: the collection itself; codewords: residuals, one Gaussian
        mix = Mixture(case["kind"] if k != 256 else "other", D, max(64, k // 4) if k != 256 else 1, seed)
        X = mix.vectors(case["nt"])
        return dict(case=case, X=X, C0=X[torch.randperm(case["nt"], generator=mix.g, device=DEV)[:k]].contiguous(),
                    C=torch.empty(k, D, device=DEV), assign=torch.empty(case["nt"], dtype=torch.int32, device=DEV),
                    counts=torch.empty(k, dtype=torch.int32, device=DEV))
    mix = Mixture(case["kind"], D, max(16, k // 4), seed)
    C, P = mix.centroids(k), mix.codewords(case["m"])
    if do == "build":
        return dict(case=case, C=C, P=P, X=mix.vectors(case["N"]))
    idx = Index(case, C, P)
    if do == "encode":
        nb = case["nb"]
        return dict(case=case, idx=idx, X=mix.vectors(nb), cell=torch.empty(nb, dtype=torch.int32, device=DEV),
                    edge=torch.empty(nb, dtype=torch.int32, device=DEV), lam=torch.empty(nb, dtype=torch.uint8, device=DEV),
                    codes=torch.empty(nb, case["m"], dtype=torch.uint8, device=DEV))
    _stored_points(case, mix, idx)
    nq, K = case["nq"], case["K"]
    return dict(case=case, idx=idx, Y=mix.vectors(nq), dist=torch.empty(nq, K, device=DEV),
                ids=torch.empty(nq, K, dtype=torch.int32, device=DEV))


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(state):
    c = state["case"]
    if c["do"] == "search":
        search = vlq.vlq_search_noalloc if c["noalloc"] else vlq.vlq_search
        search(state["idx"].h, state["Y"], c["nq"], c["w1"], c["w2"], c["K"], state["dist"], state["ids"])
        return state["dist"], state["ids"]
    if c["do"] == "encode":
        out = state["cell"], state["edge"], state["lam"], state["codes"]
        vlq.vlq_encode(state["idx"].h, state["X"], c["nb"], *out)
        return out
    if c["do"] == "train":
        state["C"].copy_(state["C0"])
        vlq.vlq_kmeans(state["X"], c["nt"], c["D"], c["k"], c["iters"], state["C"], state["assign"], state["counts"])
        return state["C"], state["assign"], state["counts"]
    idx = Index(c, state["C"], state["P"], state["X"])
    k, n, m, N = c["k"], c["n"], c["m"], c["N"]
    S, E = torch.empty(k, n, dtype=torch.int32, device=DEV), torch.empty(k, n, device=DEV)
    off = torch.empty(k * n + 1, dtype=torch.int64, device=DEV)
    ids, lam = torch.empty(N, dtype=torch.int32, device=DEV), torch.empty(N, dtype=torch.uint8, device=DEV)
    codes = torch.empty(N, m, dtype=torch.uint8, device=DEV)
    vlq.vlq_index_get_graph(idx.h, S, E)
    vlq.vlq_index_get_lists(idx.h, off, ids, codes, lam)
    idx.close()
    return S, E, off, ids, codes, lam


def work(case):
    """What a pass cannot do without: every input read once, every output written once, and the method's own
    multiply-adds (one distance per pair it compares, m table entries added per scanned point)."""
    k, D = case["k"], case["D"]
    if case["do"] == "train":
        nt, sweeps = case["nt"], case["iters"] + 1
        return {"bytes": sweeps * 4 * nt * D + 4 * (2 * k * D + nt + k), "flops": sweeps * 2 * nt * k * D}
    n, m = case["n"], case["m"]
    books = 4 * (k * D + 256 * D)
    one_encode = 2 * k * D + 2 * n * D + 2 * 256 * D
    if case["do"] == "encode":
        nb = case["nb"]
        return {"bytes": books + 8 * k * n + nb * (4 * D + 9 + m), "flops": nb * one_encode}
    N = case["N"]
    if case["do"] == "build":
        return {"bytes": books + N * (4 * D + 2 * (m + 9)) + 16 * k * n, "flops": N * one_encode + 2 * k * k * D}
    nq, w1, w2, K = (case[x] for x in ("nq", "w1", "w2", "K"))
    scanned = nq * w2 * N / (k * n)  # points; those of one list count once for the bytes
    return {"bytes": books + min(scanned, N) * (m + 5) + 8 * min(nq * w1, k) * n + nq * (4 * D + 12 * K),
            "flops": 2 * nq * (k + w1 * n + 256) * D + scanned * m}


def tolerance(case):
    if case["do"] == "search":
        # the scan against the one with 2m lookups, i.e. other sums of the same fp32 terms: 1.3e-7, 4.5e-7, 4e-5
        return {"rel": 1e-6, "max": 2e-6, "differ": 2e-4}
    if case["do"] == "train":
        # against Lloyd in 64 bits: 2.5e-8, 6e-8, no vector elsewhere; one vector that is within a rounding of two
        # centroids and goes to the other moves a single centroid by a few per cent
        return {"rel": 1e-4, "max": 2e-2, "differ": 1e-5}
    if case["do"] == "encode":
        # fp32 contraction and another summation order of the line distances: 2e-6
        return {"differ": 1e-5}
    # a point that goes to another list moves the places of those between the two lists
    return {"rel": 1e-6, "max": 1e-5, "differ": 1e-3}
