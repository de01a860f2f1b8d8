"""A ray's composite and gradients are the same bits whichever rays are beside it:
rays of up to 16 samples among themselves, where a wave takes one sample a lane,
and next to longer rays, where it takes four (which other tests compare with the
oracle)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api

pytestmark = pytest.mark.gpu
TOL = 1e-4


def _inputs(counts, rng):
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(off[-1])
    t0 = rng.uniform(2.0, 6.0, n).astype(np.float32)
    t1 = (t0 + rng.uniform(0.0, 0.02, n)).astype(np.float32)
    sigma = np.exp(3.0 * rng.normal(size=n)).astype(np.float32)
    return (off, t0, t1, sigma, rng.random((n, 3)).astype(np.float32),
            rng.normal(size=(counts.size, 3)).astype(np.float32), rng.normal(size=counts.size).astype(np.float32))


def _run(x):
    dev = [torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in x]
    C, A = api.composite_forward(*dev[:5])
    ds, dc = api.composite_backward(*dev)
    return [v.cpu().numpy() for v in (C, A, ds, dc)]


@pytest.mark.parametrize("beside", [17, 64, 65, 128, 129, 300])
@pytest.mark.parametrize("most", [1, 4, 5, 15, 16])
def test_short_rays_beside_long_ones(most, beside):
    rng = np.random.default_rng(9900 + most)
    n = 401
    short = rng.integers(0, most + 1, n)
    short[::7] = most
    counts = np.stack([short, np.full(n, beside)], 1).reshape(-1)
    both = _inputs(counts, rng)
    own = np.repeat(np.arange(2 * n) % 2 == 0, counts)
    alone = (np.concatenate([[0], np.cumsum(short)]).astype(np.int64), *(v[own] for v in both[1:5]), both[5][::2], both[6][::2])
    got, want = _run(both), _run(alone)
    for a, b in zip((got[0][::2], got[1][::2], got[2][own], got[3][own]), want):
        np.testing.assert_array_equal(a, b)
    # the pixels and the colours' gradients, whose sums do not cancel, also against the oracle
    off, t0, t1, sigma, rgb, g_rgb, g_a = both
    C, A, _ = oracle.composite_forward_all(off, t0, t1, sigma, rgb)
    _, dc = oracle.composite_backward_all(off, t0, t1, sigma, rgb, g_rgb, g_a)
    assert (np.abs(got[0] - C).max(1) <= TOL * np.maximum(np.abs(C).max(1), 1e-30)).all()
    assert (np.abs(got[1] - A) <= TOL * np.maximum(A, 1e-30)).all()
    assert np.abs(got[3] - dc).max() <= TOL * np.abs(dc).max()
