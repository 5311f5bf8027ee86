"""The error bound of the encoder's fp16 product (Alg. 1, nearest centroid), checked on the CPU in fp64: images as the
kernel writes them (a power-of-two scale per block, round to nearest even, values below 2^-14 as zero), the residual
norms that the bound is made of, and the band of a row against every column's true distance."""
import numpy as np
import pytest


def image(V):
    m = np.abs(V).max()
    ex = 14 - int(np.floor(np.log2(m))) if m > 0 else 0
    s = 2.0 ** max(-60, min(60, ex))
    q = (V.astype(np.float32) * np.float32(s)).astype(np.float16).astype(np.float64)
    q[np.abs(q) < 2.0 ** -14] = 0.0
    return q / s


def band(na, res, rho, big, dmin, D):
    if not res <= 2.0 ** -9 * na:
        return np.inf
    s = 1.1 * (na + np.sqrt(dmin)) + 1.5 * np.sqrt(na * big)
    return 4 * ((res + 1.01 * rho * na) * s + 1.01 * na * big) + 8 * (D + 8) * 2.0 ** -24 * s * s


@pytest.mark.parametrize("D", [32, 96, 128])
@pytest.mark.parametrize("kind", ["real", "integer", "wide", "aligned", "tiny_column", "far_row"])
def test_band_holds_the_true_nearest(kind, D):
    rng = np.random.default_rng(D + len(kind))
    for trial in range(20):
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
        A, B = A.astype(np.float32).astype(np.float64), B.astype(np.float32).astype(np.float64)
        Ai, Bi = image(A), image(B)
        ra, rb = np.linalg.norm(A - Ai, axis=1) * 1.0001, np.linalg.norm(B - Bi, axis=1) * 1.0001
        na, nb = np.linalg.norm(A, axis=1), np.linalg.norm(B, axis=1)
        small = rb <= 5e-4 * nb
        rho, big = (rb[small] / nb[small]).max(initial=0.0) * 1.0001, rb[~small].max(initial=0.0)
        if kind == "integer":
            assert (ra == 0).all()
        approx = nb ** 2 - 2 * Ai @ Bi.T
        true = ((A[:, None] - B[None]) ** 2).sum(2)
        # the bound itself
        assert (np.abs(A @ B.T - Ai @ Bi.T) <= ra[:, None] * nb + 1.002 * na[:, None] * np.maximum(rho * nb, big) + 1e-12 * na[:, None] * nb).all()
        # and what it is for: the true nearest column is inside the band of the smallest approximate value
        for i in range(len(A)):
            dmin = max(approx[i].min() + na[i] ** 2, 0.0)
            assert approx[i, true[i].argmin()] <= approx[i].min() + band(na[i], ra[i], rho, big, dmin, D)


def test_band_is_not_vacuous():
    """Vectors built to align every rounding error come within a factor of the bound on the product."""
    a = np.full((1, 128), 1 + 2.0 ** -11 - 2.0 ** -22)
    err = abs((a @ a.T - image(a) @ image(a).T).item())
    assert err > 0.9 * 2 * np.linalg.norm(a - image(a)) * np.linalg.norm(a)
