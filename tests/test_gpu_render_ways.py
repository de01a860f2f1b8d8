"""The render's two ways of sharing a wave's rays among its rows: equal lengths
(a ray a row), lengths so uneven that their chunks are dealt out, and waves of
each next to one another, from one blob to sixteen and at both numbers of rays
a wave.  Per ray within 1e-4 of the float64 oracle, as every render test."""
import numpy as np
import pytest

from tests.test_gpu_render_chunks import _check, _field, _rays, _steps

pytestmark = pytest.mark.gpu


def _counts(kind, n, rng):
    if kind == "short":
        return rng.integers(0, 17, n)
    if kind == "equal":
        return np.full(n, 3 * 16 + 5)
    if kind == "uneven":
        return np.where(rng.random(n) < 0.2, rng.integers(200, 600, n), rng.integers(0, 3, n))
    # around the line between the ways: one of eight rays longer and longer
    return np.where(np.arange(n) % 8 == 5, 16 * (np.arange(n) // 8 % 24), 20)


@pytest.mark.parametrize("blobs", [1, 4, 5, 12, 16])
@pytest.mark.parametrize("kind", ["short", "equal", "uneven", "line"])
def test_ways_of_sharing_rows(kind, blobs):
    rng = np.random.default_rng(9550 + blobs)
    for n in (1, 6, 803):
        counts = _counts(kind, n, rng)
        counts[0] = max(counts[0], 1)    # some sample
        _check(counts, *_rays(n, rng), *_steps(int(counts.sum()), rng), _field(blobs, rng))


@pytest.mark.parametrize("kind", ["short", "line"])
def test_ways_with_eight_rays_a_wave(kind):
    rng = np.random.default_rng(9560)
    n = 524288 + 11
    counts = _counts(kind, n, rng)
    counts[4000:-4000] = np.minimum(counts[4000:-4000], 1)
    _check(counts, *_rays(n, rng), *_steps(int(counts.sum()), rng), _field(6, rng))
