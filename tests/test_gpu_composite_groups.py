"""The composite's groups of four samples and chunks of 64 at their edges:
ray lengths around them, groups that run into the next ray or to the last
sample of the arrays, samples no ray owns (NaN, which must not reach any
output), thin and thick samples on both sides of the switch between the series
and the exponential.  Per ray within 1e-4 of the float64 oracle, the bound of
every composite test."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api

pytestmark = pytest.mark.gpu

TOL = 1e-4
LENGTHS = [0, 1, 2, 3, 4, 5, 15, 16, 17, 60, 61, 63, 64, 65, 68, 127, 128, 129, 191, 257, 3, 1]


def _packed(order, head, tail, depth, rng):
    counts = np.asarray(LENGTHS)[rng.permutation(len(LENGTHS))] if order == "mixed" else np.asarray(LENGTHS)
    off = head + np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    n = int(off[-1]) + tail
    t0 = np.sort(rng.uniform(2.0, 6.0, n)).astype(np.float32)
    dt = rng.uniform(0.004, 0.006, n).astype(np.float32)
    t1 = (t0 + dt).astype(np.float32)
    # optical depths per sample: thin, around one half, or thick
    tau = {"thin": rng.uniform(0.0, 0.05, n), "half": 0.5 + rng.uniform(-1e-3, 1e-3, n),
           "thick": np.exp(rng.uniform(-6.0, 3.0, n)) * rng.integers(0, 2, n)}[depth]
    sigma = (tau / (t1 - t0).astype(np.float64)).astype(np.float32)
    rgb = rng.random((n, 3)).astype(np.float32)
    own = np.zeros(n, bool)
    own[off[0]:off[-1]] = True
    for x in (t0, t1, sigma, rgb):
        x[~own] = np.nan
    return off, t0, t1, sigma, rgb, own


def _close(got, ref, what):
    err = np.abs(got.astype(np.float64) - ref).max(initial=0.0)
    assert err <= TOL * max(np.abs(ref).max(initial=0.0), 1e-30), (what, err)


@pytest.mark.parametrize("depth", ["thin", "half", "thick"])
@pytest.mark.parametrize("head,tail", [(0, 0), (3, 0), (0, 1), (5, 7)])
def test_groups_and_chunks_at_their_edges(head, tail, depth):
    rng = np.random.default_rng(9400 + 10 * head + tail)
    off, t0, t1, sigma, rgb, own = _packed("mixed" if head else "sorted", head, tail, depth, rng)
    n = len(off) - 1
    g_rgb, g_a = rng.normal(size=(n, 3)).astype(np.float32), rng.normal(size=n).astype(np.float32)
    dev = [torch.from_numpy(x).cuda() for x in (off, t0, t1, sigma, rgb)]
    C, A = (x.cpu().numpy() for x in api.composite_forward(*dev))
    ds, dc = (x.cpu().numpy() for x in api.composite_backward(*dev, torch.from_numpy(g_rgb).cuda(),
                                                               torch.from_numpy(g_a).cuda()))
    z = off - off[0]
    s = slice(off[0], off[-1])
    Cr, Ar, _ = oracle.composite_forward_all(z, t0[s], t1[s], sigma[s], rgb[s])
    dsr, dcr = oracle.composite_backward_all(z, t0[s], t1[s], sigma[s], rgb[s], g_rgb, g_a)
    for r in range(n):
        a, b = z[r], z[r + 1]
        _close(C[r], Cr[r], ("rgb", r))
        _close(A[r], Ar[r], ("opacity", r))
        _close(ds[s][a:b], dsr[a:b], ("d_sigma", r))
        _close(dc[s][a:b], dcr[a:b], ("d_rgb", r))
    assert not ds[~own].any() and not dc[~own].any()
