"""CPU test of the strip spheres' scale: pixels per unit of length at most, over a bounding sphere.

With a = h (row x + row w), b = row w, the window position of v is x(v) = (a . v + a3) / (b . v + b3).  Over a
ball of radius p around c, with x0 = x(c), w0 = w(c) and w1 = w0 - p |b| > 0, any two points satisfy
|x(u) - x(v)| <= L |u - v|, L = |a - x0 b| (1 + p |b| / w1) / w1."""
import numpy as np
import pytest


@pytest.mark.parametrize("nearness", [0.01, 0.1, 0.28, 0.6, 0.95])
def test_scale_bounds_projected_distances(nearness):
    rng = np.random.default_rng(int(100 * nearness))
    for _ in range(200):
        a, b = rng.normal(size=3) * 10.0 ** rng.uniform(-2, 3), rng.normal(size=3) * 10.0 ** rng.uniform(-1, 1)
        c = rng.normal(size=3)
        p = 10.0 ** rng.uniform(-3, 1)
        w0 = p * np.linalg.norm(b) / nearness
        b3 = w0 - b @ c
        a3 = rng.uniform(-1, 3) * 500 * w0 - a @ c
        w1 = w0 - p * np.linalg.norm(b)
        x0 = (a @ c + a3) / w0
        L = np.linalg.norm(a - x0 * b) * (1 + p * np.linalg.norm(b) / w1) / w1
        d = rng.normal(size=(2, 64, 3))
        d *= (p * rng.uniform(0, 1, (2, 64, 1)) ** 0.2) / np.linalg.norm(d, axis=2, keepdims=True)
        d[0, 0] = -p * b / np.linalg.norm(b)          # the nearest point of the ball
        v = c + d
        x = (v @ a + a3) / (v @ b + b3)
        gap = np.abs(x[0] - x[1]) - L * np.linalg.norm(d[0] - d[1], axis=1)
        assert (gap <= 1e-9 * np.abs(x).max()).all(), gap.max()
