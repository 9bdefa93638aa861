"""CPU check of the per-draw margin of the stage-1 fast path: window positions as the kernels compute
them (prescaled rows of interior draws, or the exact transform with a reciprocal one ulp off) stay within
the margin of the snapped positions of the exact path, for random cameras, placements and view sizes."""
import math

import numpy as np
import pytest

f32 = np.float32
U = 2.0 ** -24


def fma(a, b, c):
    return f32(np.float64(a) * np.float64(b) + np.float64(c))


def row(A, v):
    return fma(A[0], v[0], fma(A[1], v[1], fma(A[2], v[2], A[3])))


def snapped(A, v, h):
    """Exact path: window position snapped to 1/256 px, in pixels, for rows (axis, w) of A."""
    x, w = row(A[0], v), row(A[1], v)
    z = f32(1.0 / np.float64(w))
    return np.rint(np.float64(fma(f32(x * z), h, h)) * 256.0) / 256.0


def rcp(w, ulps):
    r = f32(1.0 / np.float64(w))
    return np.nextafter(r, f32(np.inf) if ulps > 0 else f32(-np.inf)) if ulps else r


def interior_margin(A, c, r, h):
    """The bound of prescaled draws over a bounding sphere (c, r), one axis, and the prescaled row."""
    A64 = A.astype(np.float64)
    S = [abs(A64[k, 3]) + sum(abs(A64[k, j]) * (abs(c[j]) + r) for j in range(3)) for k in (0, 1)]
    g = np.linalg.norm(A64[1, :3])
    mag = abs(A64[1, 3]) + np.abs(A64[1, :3] * c).sum()
    w_lo = A64[1, 3] + A64[1, :3] @ c - r * g - 1e-4 * (mag + r * g)
    if w_lo <= 0:
        return None, None
    m = 1.01 * (h * U * ((7 * S[0] + 19 * S[1]) / w_lo + 16) + (3 * h + 1) * U) + 2.0 ** -9
    return m, (h * (A64[0] + A64[1])).astype(f32)


@pytest.mark.parametrize("size", [1, 17, 256, 1920, 16384])
def test_fast_positions_stay_within_the_margin(size):
    rng = np.random.default_rng(size)
    h = f32(size / 2)
    checked = [0, 0]
    worst = [0.0, 0.0]
    for _ in range(4000):
        scale = 10 ** rng.uniform(-4, 2)                       # object units per world unit
        q, _ = np.linalg.qr(rng.normal(size=(3, 3)))
        A = np.empty((2, 4))
        f = 10 ** rng.uniform(-0.3, 0.7)
        A[0, :3], A[1, :3] = q[0] * f * scale, q[1] * scale
        depth = 10 ** rng.uniform(-1, 2)
        r = rng.uniform(1e-4, 0.3) * depth / scale
        c = rng.normal(size=3) * r * 10 ** rng.uniform(-1, 1)  # centres up to ten radii off the origin
        A[0, 3] = rng.uniform(-1, 1) * depth - A[0, :3] @ c
        A[1, 3] = depth - A[1, :3] @ c
        A = A.astype(f32)
        m_in, R = interior_margin(A, c, r, float(h))
        m_gen = 1.01 * (1.625 * math.ldexp(float(h), -20) + math.ldexp(3 * float(h) + 1, -23)) + 2.0 ** -9
        for _ in range(3):
            d = rng.normal(size=3)
            v = (c + d / np.linalg.norm(d) * r * rng.uniform(0, 1) ** (1 / 3)).astype(f32)
            x, w = row(A[0], v), row(A[1], v)
            if not w >= 0.01 or abs(x) > 1.99 * w:
                continue
            exact = snapped(A, v, h)
            t = rcp(w, rng.integers(-1, 2))
            general = np.float64(fma(f32(x * t), h, h))
            checked[0] += 1
            worst[0] = max(worst[0], abs(general - exact) / m_gen)
            if m_in is not None and m_in <= 1 / 32:
                fast = np.float64(f32(row(R, v) * t))
                checked[1] += 1
                worst[1] = max(worst[1], abs(fast - exact) / m_in)
    assert checked[0] > 2000 and checked[1] > 1000, checked
    assert worst[0] <= 1.0 and worst[1] <= 1.0, worst
