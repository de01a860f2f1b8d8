"""The blob-field render at the edges of its work split: ray counts around a
wave's share at each of its sizes, ray lengths around chunks of 16, waves of
empty rays, one ray that fills a whole wave's ranges, every number of blobs,
directions that are not unit, tiny or zero.  Per ray within 1e-4 of the float64
oracle, as every render test."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api

pytestmark = pytest.mark.gpu

TOL = 1e-4


def _field(k, rng):
    return (rng.uniform(-0.7, 0.7, (k, 3)).astype(np.float32), rng.uniform(0.2, 0.5, k).astype(np.float32),
            rng.uniform(5.0, 40.0, k).astype(np.float32), rng.random((k, 3)).astype(np.float32))


def _check(counts, o, d, t0, t1, blobs):
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    dev = [torch.from_numpy(x).cuda() for x in (off, o, d, t0, t1)]
    C, A = (x.cpu().numpy() for x in api.render_blobs(*dev, api.blob_field(*blobs)))
    Cr, Ar = oracle.render_blobs_all(off, o, d, t0, t1, *blobs)
    bad = np.abs(C - Cr).max(axis=1) > TOL * np.maximum(np.abs(Cr).max(axis=1), 1e-30)
    assert not bad.any(), (np.nonzero(bad)[0][:5], C[bad][:2], Cr[bad][:2])
    bad = np.abs(A - Ar) > TOL * np.maximum(np.abs(Ar), 1e-30)
    assert not bad.any(), (np.nonzero(bad)[0][:5], A[bad][:2], Ar[bad][:2])


def _rays(n, rng, length=1.0):
    d = rng.normal(size=(n, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    o = rng.uniform(-0.3, 0.3, (n, 3)) - 4.0 * d
    return o.astype(np.float32), (d * length).astype(np.float32)


def _steps(n, rng, length=1.0):
    t0 = rng.uniform(3.0, 5.0, n) / length
    return t0.astype(np.float32), (t0 + rng.uniform(0.003, 0.02, n) / length).astype(np.float32)


@pytest.mark.parametrize("blobs", range(1, 17))
def test_every_number_of_blobs_and_lengths_around_chunks(blobs):
    rng = np.random.default_rng(9500 + blobs)
    lengths = np.asarray([0, 1, 2, 15, 16, 17, 31, 32, 33, 63, 64, 65, 250, 0, 0, 3])
    for n in (1, 3, 4, 5, 17, 64, 67):
        counts = rng.choice(lengths, n)
        counts[rng.integers(0, n)] = 40
        _check(counts, *_rays(n, rng), *_steps(int(counts.sum()), rng), _field(blobs, rng))


@pytest.mark.parametrize("n", [131071, 131072, 262143, 262144, 262161, 524287, 524288, 524297])
def test_ray_counts_around_the_waves_shares(n):
    rng = np.random.default_rng(9520)
    counts = rng.choice([0, 0, 1, 2, 7, 20], n)
    counts[100:140] = 0
    counts[-3] = 900          # one ray over every range of the last wave
    _check(counts, *_rays(n, rng), *_steps(int(counts.sum()), rng), _field(5, rng))


@pytest.mark.parametrize("length", [1e-20, 0.01, 37.0, 1e12])
def test_directions_of_any_length(length):
    rng = np.random.default_rng(9530)
    counts = rng.integers(0, 50, 40)
    o, d = _rays(40, rng, length)
    t0, t1 = _steps(int(counts.sum()), rng, length)
    _check(counts, o, d, t0, t1, _field(7, rng))


def test_still_rays():
    """A zero direction samples the field at its origin."""
    rng = np.random.default_rng(9540)
    counts = rng.integers(0, 40, 20)
    o, d = _rays(20, rng)
    o, d = rng.uniform(-0.5, 0.5, (20, 3)).astype(np.float32), np.zeros_like(d)
    _check(counts, o, d, *_steps(int(counts.sum()), rng), _field(12, rng))
