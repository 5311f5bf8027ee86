"""The error bound of the encoder's fp16 product (Alg. 1, nearest centroid), checked on the CPU: images as the kernel writes
them (round to nearest even, values below 2^-14 as zero), products added up in fp32, keys with the tile's index planted,
and the band of a row (nn_half_band and what goes into it, compiled from csrc/bounds.h) against every column's true distance."""
import numpy as np
import pytest

import host_bounds

f32 = np.float32


def round_half(V, ex):
    """V at the scales 2^ex, as fp16, and scaled back (exactly)"""
    s = 2.0 ** np.asarray(ex, np.float64)
    q = (V * s).astype(f32).astype(np.float16).astype(np.float64)
    q[np.abs(q) < 2.0 ** -14] = 0.0
    return q / s


def row_image(V, host):
    ex = host.exponent_of(np.abs(V).max())
    own = np.array([[host.exponent_of(m)] for m in np.abs(V).max(1)])
    lost = (np.abs(V).max(1) > 0) & (own[:, 0] > ex + host.gap())
    return round_half(V, own if lost.any() else ex)


def column_image(V, host):
    return round_half(V, host.exponent_of(np.abs(V).max()))


def norm2(V):
    """squared norms, added up in fp32"""
    s = np.zeros(len(V), f32)
    for d in range(V.shape[1]):
        s = (V[:, d] ** 2 + s).astype(f32)
    return s


def keys(Ai, Bi, nb2, bits, rng):
    """||b||^2 - 2 <a', b'>: products exact (22 bits), sums in fp32, then the low bits replaced by a tile's index"""
    acc = np.zeros((len(Ai), len(Bi)), f32)
    for d in range(Ai.shape[1]):
        acc = (acc + Ai[:, None, d] * Bi[None, :, d]).astype(f32)
    e = (nb2.astype(np.float64) - 2.0 * acc).astype(f32)
    low = np.uint32((1 << bits) - 1)
    u = (e.view(np.uint32) & ~low) | rng.integers(0, 1 << bits, e.shape, dtype=np.uint32)
    return u.view(f32), (u & ~low).view(f32)


@pytest.mark.parametrize("D", [32, 96, 128])
@pytest.mark.parametrize("kind", ["real", "integer", "wide", "aligned", "tiny_column", "far_row", "small_rows", "groups"])
def test_band_holds_the_true_nearest(kind, D):
    host = host_bounds.lib()
    rng = np.random.default_rng(D + len(kind))
    bits = host.idx_bits(512)  # 65 536 columns in one split: the widest index
    assert bits == 9
    for trial in range(10):
        A = rng.normal(size=(32, D))
        B = np.concatenate([A + rng.normal(scale=10.0 ** rng.uniform(-6, 0), size=A.shape) for _ in range(4)])
        if kind == "integer":
            A, B = np.rint(A * 60), B * 60
        elif kind == "wide":
            A, B = (x * np.exp(rng.normal(scale=4.0, size=x.shape)) for x in (A, B))
        elif kind == "aligned":  # every component just below a rounding boundary of 11 bits
            A = (1 + 2.0 ** -11 - 2.0 ** -22) * 2.0 ** rng.integers(-3, 4, A.shape)
            B = (1 + 2.0 ** -11 - 2.0 ** -22) * 2.0 ** rng.integers(-3, 4, B.shape)
        elif kind == "tiny_column":
            B[3] *= 1e-9
            B[5] *= 1e4
        elif kind == "far_row":
            A[7] *= 1e6
        elif kind == "small_rows":
            A[::2] *= 10.0 ** rng.uniform(-9, -4, (16, 1))
        elif kind == "groups":
            B = np.repeat(rng.normal(size=(8, D)), 16, 0) + 0.02 * rng.normal(size=(128, D))
            A = B[rng.integers(0, 128, 32)] + 0.3 * rng.normal(size=A.shape)
        A, B = A.astype(f32).astype(np.float64), B.astype(f32).astype(np.float64)
        Ai, Bi = row_image(A, host), column_image(B, host)
        ra, rb = np.linalg.norm(A - Ai, axis=1) * 1.0001, np.linalg.norm(B - Bi, axis=1) * 1.0001
        na, nb = np.linalg.norm(A, axis=1), np.linalg.norm(B, axis=1)
        assert (ra <= 1.01 * 2.0 ** -11 * na).all()  # no row loses more than the rounding
        small = rb <= host.rel_max() * nb
        rho, big = (rb[small] / nb[small]).max(initial=0.0) * 1.0001, rb[~small].max(initial=0.0)
        if kind == "integer":
            assert (ra == 0).all()
        # the bound on a product itself
        bound = ra[:, None] * nb + 1.002 * na[:, None] * np.maximum(rho * nb, big) + 1e-12 * na[:, None] * nb
        assert (np.abs(A @ B.T - Ai @ Bi.T) <= bound).all()
        # and what it is for: the true nearest column is inside the band of the smallest key
        an2, nb2 = norm2(A), norm2(B)
        planted, e = keys(Ai, Bi, nb2, bits, rng)
        true = ((A[:, None] - B[None]) ** 2).sum(2)
        for i in range(len(A)):
            emin = e[i, planted[i].argmin()]
            dmin = max(emin + an2[i], f32(0))
            band = host.half_band(an2[i], ra[i], rho, big, dmin, host.band_dist(bits), D)
            assert e[i, true[i].argmin()] <= emin + f32(band)
            if kind in ("real", "integer", "groups"):  # (and the band is not simply everything)
                assert band < 4e-3 * (an2[i] + true[i].min()) * 4


def test_band_is_not_vacuous():
    """Vectors built to align every rounding error come within a factor of the bound on the product."""
    host = host_bounds.lib()
    a = np.full((1, 128), 1 + 2.0 ** -11 - 2.0 ** -22)
    ai = row_image(a, host)
    err = abs((a @ a.T - ai @ ai.T).item())
    assert err > 0.9 * 2 * np.linalg.norm(a - ai) * np.linalg.norm(a)


@pytest.mark.parametrize("bits", [1, 5, 9, 18])
def test_planting_is_covered(bits):
    """Half of band_dist covers what the planted bits can move a key by (the minimum's and the candidate's)."""
    host = host_bounds.lib()
    rng = np.random.default_rng(bits)
    e = (rng.normal(size=100_000) * 10.0 ** rng.uniform(-5, 5, 100_000)).astype(f32)
    low = np.uint32((1 << bits) - 1)
    for planted in (e.view(np.uint32) & ~low, e.view(np.uint32) | low):
        moved = np.abs(planted.view(f32).astype(np.float64) - e) / np.abs(e)
        assert moved.max() <= host.band_dist(bits) / 2
    assert moved.max() > host.band_dist(bits) / 10


@pytest.mark.parametrize("D", [32, 64, 96, 128])
def test_accumulation_is_covered(D):
    """Twice the error of the fp32 sums (norm, product, their difference) against what the band has for it alone."""
    host = host_bounds.lib()
    rng = np.random.default_rng(D)
    worst = 0.0
    for trial in range(50):
        a = round_half(np.abs(rng.normal(size=(1, D))) + 1, 11).astype(f32).astype(np.float64)
        b = round_half(np.abs(rng.normal(size=(64, D))) + 1, 11).astype(f32).astype(np.float64)
        _, e = keys(a, b, norm2(b), 0, rng)
        err = np.abs(e[0] - ((b ** 2).sum(1) - 2 * (b @ a[0]))).max()
        na2 = (a ** 2).sum()
        d = ((a - b) ** 2).sum(1).min()
        band = host.half_band(na2, 0, 0, 0, d, 0, D)
        assert 2 * err <= band
        worst = max(worst, 2 * err / band)
    assert worst > 1e-3


@pytest.mark.parametrize("D", [32, 64, 96, 128])
def test_accumulation_onto_the_norm_is_covered(D):
    """The kernel's own order: half the norm first, the products added to it."""
    host = host_bounds.lib()
    rng = np.random.default_rng(D + 1)
    worst = 0.0
    for trial in range(50):
        a = round_half(np.abs(rng.normal(size=(1, D))) + 1, 11)
        b = round_half(np.abs(rng.normal(size=(64, D))) + 1, 11)
        if trial % 2:  # all of one sign: the partial sums grow to |b|^2 / 2 + |a||b|
            a = -a
        acc = (0.5 * norm2(b)).astype(f32)
        for d in range(D):
            acc = (acc - a[0, d] * b[:, d]).astype(f32)
        err = np.abs(2.0 * acc.astype(np.float64) - ((b ** 2).sum(1) - 2 * (b @ a[0]))).max()
        d = ((a - b) ** 2).sum(1).min()
        band = host.half_band((a ** 2).sum(), 0, 0, 0, d, 0, D)
        assert 2 * err <= band
        worst = max(worst, 2 * err / band)
    assert worst > 1e-3


def test_lossy_columns_are_covered():
    """A column that lost `big` of itself moves a product by up to |a'| big, twice in each of two values."""
    host = host_bounds.lib()
    for na, big in ((1.0, 1e-3), (30.0, 2.0), (1e-3, 5.0)):
        assert host.half_band(na * na, 0, 0, big, 0.5, 0, 128) - host.half_band(na * na, 0, 0, 0, 0.5, 0, 128) >= 4 * na * big
