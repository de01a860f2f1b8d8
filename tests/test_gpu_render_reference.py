"""Rendering through fields that are not compact: one blob or most blobs far
from the others, with density and without.  Per ray within 1e-4 of the float64
oracle, the bound of every render test."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api

pytestmark = pytest.mark.gpu
TOL = 1e-4


def _case(rng, n=500, length=120, radius=4.0):
    dirs = rng.normal(size=(n, 3))
    dirs /= np.linalg.norm(dirs, axis=1, keepdims=True)
    aim = rng.uniform(-0.6, 0.6, (n, 3))
    o = (aim - radius * dirs).astype(np.float32)
    k = np.tile(np.arange(length), n)
    first = np.float32(radius - 1.5)
    t0 = (first + k * np.float32(0.025)).astype(np.float32)
    t1 = (first + (k + 1) * np.float32(0.025)).astype(np.float32)
    return np.arange(n + 1, dtype=np.int64) * length, o, dirs.astype(np.float32), t0, t1


def _blobs(rng, k=12):
    return [rng.uniform(-0.7, 0.7, (k, 3)), rng.uniform(0.2, 0.5, k), rng.uniform(5.0, 40.0, k), rng.random((k, 3))]


def _check(off, o, d, t0, t1, blobs, tol=TOL):
    blobs = [np.asarray(b, np.float32) for b in blobs]
    C, A = api.render_blobs(*(torch.from_numpy(x).cuda() for x in (off, o, d, t0, t1)), api.blob_field(*blobs))
    Cr, Ar = oracle.render_blobs_all(off, o, d, t0, t1, *blobs)
    assert (Ar > 1e-2).mean() > 0.5
    err = np.abs(C.cpu().numpy() - Cr).max(1) / np.maximum(np.abs(Cr).max(1), 1e-30)
    err_a = np.abs(A.cpu().numpy() - Ar) / np.maximum(Ar, 1e-30)
    assert max(err.max(), err_a.max()) <= tol, (float(err.max()), float(err_a.max()))


@pytest.mark.parametrize("density", [0.0, 20.0])
@pytest.mark.parametrize("distance", [10.0, 1e3, 1e5, 1e6, 1e8])
def test_one_blob_far_from_the_others(distance, density):
    rng = np.random.default_rng(9860)
    off, o, d, t0, t1 = _case(rng)
    blobs = _blobs(rng)
    blobs[0][-1] = distance * np.asarray([0.6, -0.48, 0.64])
    blobs[2][-1] = density
    _check(off, o, d, t0, t1, blobs)


def test_most_blobs_far():
    rng = np.random.default_rng(9861)
    off, o, d, t0, t1 = _case(rng)
    blobs = _blobs(rng)
    blobs[0][4:] *= 1e6
    _check(off, o, d, t0, t1, blobs)
