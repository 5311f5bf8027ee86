"""Arithmetic that kernels rely on (csrc/bounds.h), compiled for the host and checked there."""
import numpy as np
import pytest

import host_bounds


@pytest.fixture(scope="module")
def host():
    return host_bounds.lib()


# an index holds up to 2^31 - 1 points: the places behind its last turn need 32 bits
@pytest.mark.parametrize("total", [1, 2047, 2048, 2049, 10_000, 2**31 - 4097, 2**31 - 2049, 2**31 - 2048, 2**31 - 2047, 2**31 - 1])
def test_places_up_to_the_largest_index(host, total):
    assert host.last_turns(total) == 0


f32 = np.float32


def fma(a, b, c):
    """One rounding to fp32 (the product of two fp32 is exact in fp64)."""
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(f32)


def chain(a, b):
    """sum of a * b over the last axis, one fused step at a time"""
    s = np.zeros(np.broadcast(a[..., 0], b[..., 0]).shape, f32)
    for d in range(a.shape[-1]):
        s = fma(a[..., d], b[..., d], s)
    return s


def total(v):
    s = np.zeros(v.shape[:-1], f32)
    for p in range(v.shape[-1]):
        s = s + v[..., p]
    return s


@pytest.mark.parametrize("kind", ["centred", "far mean", "tight", "long edges", "small codes"])
@pytest.mark.parametrize("D,m", [(8, 8), (128, 8), (96, 16), (100, 20), (1024, 64)])
def test_fast_distance_within_slack(host, kind, D, m):
    """The one-table distance and the 2m-lookup distance of the scan, both emulated in fp32 operation by operation."""
    rng = np.random.default_rng(D + m + len(kind))
    n, ds = 400, D // m
    scale = {"tight": 0.02}.get(kind, 0.5)
    offset = {"far mean": 30.0, "tight": 3.0}.get(kind, 0.0)
    mu = (offset + rng.normal(size=D)).astype(f32)
    y = rng.normal(size=D).astype(f32)
    c = (y + scale * rng.normal(size=(n, D))).astype(f32)
    s = (c + (5 if kind == "long edges" else 1) * scale * rng.normal(size=(n, D))).astype(f32)
    w = ((1e-3 if kind == "small codes" else 0.7) * scale * rng.normal(size=(n, m, ds))).astype(f32)
    byte = rng.integers(0, 256, n)
    step64, zero = 2.0 / 255, f32(rng.uniform(0, 127))
    step = f32(step64)
    # shared by both: a, c, g (any summation order will do for the first two; g is the same number in both)
    a = chain(y - c, y - c)
    cc = chain(s - c, s - c)
    g = chain(y - c, s - c)
    sub = lambda v: v.reshape(v.shape[:-1] + (m, ds))  # noqa: E731
    # s_x in fp64, rounded once
    lh = (byte - np.float64(zero)) * step64
    c64, s64, w64 = c.astype(np.float64), s.astype(np.float64), w.astype(np.float64).reshape(n, D)
    q1 = (c64 - mu) + lh[:, None] * (s64 - c64)
    sx = ((w64 ** 2).sum(1) + 2 * (q1 * w64).sum(1) + (lh * lh - lh) * ((s64 - c64) ** 2).sum(1)).astype(f32)
    l = (byte.astype(f32) - zero) * step  # noqa: E741
    ts = total(f32(2) * chain(sub(y - mu)[None], w))
    fast = (sx - ts) + (l * fma(f32(-2) * np.ones_like(g), g, cc) + a)
    t = sub(y - c) - w
    sa, sb = total(chain(t, t)), total(chain(sub(s - c), w))
    full = fma(l, fma(l, cc, f32(2) * (sb - g)), sa)
    Q2 = total((chain(w, w)).max(0)[None])[0]
    L = max(abs(zero), abs(f32(255) - zero)) * step
    slack = host.slack(a.max(), chain(y - mu, y - mu), Q2, cc.max(), L, D, m)
    diff = np.abs(fast.astype(np.float64) - full.astype(np.float64)).max()
    assert diff <= slack
    assert slack < 3000 * diff  # (rounding errors are random, the bound adds them all up: a factor sqrt(D) and more)
