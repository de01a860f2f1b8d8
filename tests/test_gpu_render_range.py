"""Rendering where sigma is far from one: directions of any length, which scale
densities and steps, down to a sigma of 1e-31, and densities whose reciprocal is
no normal number.  Per ray within 1e-4 of the float64 oracle, the bound of every
render test."""
import numpy as np
import pytest

from tests.test_gpu_render_reference import _blobs, _case, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1e-3, 0.25, 8.0, 1024.0, 2.0 ** 107])
def test_directions_of_any_length(scale):
    rng = np.random.default_rng(9862)
    off, o, d, t0, t1 = _case(rng)
    s = np.float32(scale)
    _check(off, o, d / s, t0 * s, t1 * s, [b if i != 2 else b / scale for i, b in enumerate(_blobs(rng))])


@pytest.mark.parametrize("density", [1e30, 9e37, 2e38])
def test_densities_near_the_end_of_the_range(density):
    rng = np.random.default_rng(9863)
    off, o, d, t0, t1 = _case(rng, n=200, length=20)
    blobs = _blobs(rng, 1)
    blobs[0][:] = 0.0
    blobs[1][:] = 1e3            # one value all over
    blobs[2][:] = density
    _check(off, o, d, t0, t1, blobs)
