"""The culling tests' arithmetic, restated in numpy, where the daughters are as large as
the tests take them, and where a start is first moved to the sphere that holds the
daughters: no line that meets a sphere is dropped, whatever way the sums are rounded."""
import numpy as np
import pytest

from tests.test_gpu_cull_blocks import _filter

BOUND = 4 * 2.0 ** -22


def _towards(rng, p, T, off):
    """Directions of lines from p that pass `off` from the centres T, towards them."""
    w = T - p
    dist = np.linalg.norm(w, axis=0)
    side = np.cross(w.T, rng.normal(size=w.T.shape)).T
    side /= np.linalg.norm(side, axis=0)
    s = np.minimum(off / dist, 1.0)
    return w / dist * np.sqrt(1.0 - s * s) + side * s


def _ball(rng, n, size):
    v = rng.normal(size=(3, n))
    return v * size * rng.uniform(0, 1, n) ** (1 / 3) / np.linalg.norm(v, axis=0)


@pytest.mark.parametrize("largest", [64.0, 256.0, 512.0])
@pytest.mark.parametrize("scale", [1.0, 0.9])
def test_large_spheres(largest, scale):
    rng = np.random.default_rng(int(largest))
    n = 200000
    p, T = _ball(rng, n, 256.0), _ball(rng, n, 512.0)
    r = np.minimum(2.0 ** rng.uniform(-8, 9, n), largest)
    f = _filter(p, _towards(rng, p, T, scale * r), T, r, float(r.max()) + 0.25, BOUND, 1.0)
    assert (f < 0).all()


@pytest.mark.parametrize("far", [300.0, 1e4, 1e6, 2.0 ** 26])
def test_starts_moved_to_the_daughters_sphere(far):
    """Starts up to `far` units from the centre, in doubles, of lines that are tangent to
    spheres that reach to 0.125 units from the sphere of 256 units."""
    rng = np.random.default_rng(int(far))
    n = 200000
    r = 2.0 ** rng.uniform(-8, 6, n)
    T = rng.normal(size=(3, n))
    T *= (255.87 - r) * rng.uniform(0, 1, n) ** (1 / 6) / np.linalg.norm(T, axis=0)
    p = rng.normal(size=(3, n))
    p *= rng.uniform(0.5, 1.0, n) * far / np.linalg.norm(p, axis=0)
    e = _towards(rng, p, T, r * rng.choice([1.0, 0.99], n))
    # as the kernels form it: the nearer root of |p + t e| = 256, none past the start
    b = (p * e).sum(0)
    g = (p * p).sum(0) - 256.0 ** 2
    disc = b * b - g * (e * e).sum(0)
    out = g > 0.0
    met = out & (b < 0.0) & (disc >= 0.0)
    assert (met | ~out | (np.linalg.norm(T - p, axis=0) <= r)).all()
    t = np.where(met, g / (np.sqrt(np.maximum(disc, 0.0)) - b), 0.0)
    f = _filter(p + t * e, e, T, r, float(r.max()) + 0.25, BOUND, 1.0)
    assert (f < 0).all()
