"""The tree's classification and numbering at the edges of their work split:
grids on both sides of the size that one workgroup numbers, nodes of every
size, sides that fill no block, and refreshes that change nothing, only leaf
bits, or the structure.  Counts against numpy, contents through the decoder
(masks, ranks) and through the walks (root and child tables, sub-blocks)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api, scenes
from tests.test_gpu_sampler import assert_same, gpu_sample

pytestmark = pytest.mark.gpu

# levels, side, node log2; mask words: 1, 1000, 1331, 1024, 1536, 64, 1, 512
GRIDS = [(1, 1, 1), (1, 160, 1), (1, 168, 1), (2, 40, 5), (3, 40, 5), (2, 100, 3), (1, 9, 1), (8, 120, 4)]


def _occupancy(L, R, rng):
    n = (R + 7) // 8
    kind = rng.integers(0, 3, (L, n, n, n))
    occ = np.repeat(np.repeat(np.repeat(kind, 8, 1), 8, 2), 8, 3)[:, :R, :R, :R]
    return np.where(occ == 2, rng.random((L, R, R, R)) < 0.5, occ).astype(np.uint8)


def _counts(occ, ilog2):
    L, R = occ.shape[:2]
    S = 1 << ilog2
    NR = -(-R // (8 * S))
    pad = np.zeros((L,) + (NR * S * 8,) * 3, np.uint8)
    pad[:, :R, :R, :R] = occ
    on = pad.reshape(L, NR, S, 8, NR, S, 8, NR, S, 8).transpose(0, 1, 4, 7, 2, 5, 8, 3, 6, 9).reshape(L * NR ** 3, S ** 3, 512)
    some, every = on.any(2), on.all(2)
    mixed = some & ~every
    node = ~(every.all(1) | (~some).all(1))
    return {"n_nodes": int(node.sum()), "n_leaves": int(mixed.sum()), "n_tiles_full": int(every[node].sum()),
            "n_tiles_empty": int((~some)[node].sum()), "n_root_tiles_full": int(every.all(1).sum()),
            "n_root_tiles_empty": int((~some).all(1).sum())}


def _check(g, occ, boxes, ilog2, rays, what):
    np.testing.assert_array_equal(g.to_dense().cpu().numpy(), occ, err_msg=what)
    info = g.info()
    assert {k: info[k] for k in _counts(occ, ilog2)} == _counts(occ, ilog2), what
    o, d = rays
    far = 4.0 * 2.0 ** occ.shape[0]
    step = {"kind": "const", "dt": 0.01, "cone": 0.0, "dt_min": 0.0}
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.0, far, step, "dense_branch")
    for variant in ("branch", "subleaf_branch"):
        assert_same(gpu_sample(g, o, d, 0.0, far, step, variant, voxel_ids=False), ref, f"{what} {variant}")


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: "x".join(map(str, g)))
def test_builds_and_refreshes(grid):
    L, R, ilog2 = grid
    rng = np.random.default_rng(9600 + R + L)
    boxes = np.asarray([[-(2.0 ** k)] * 3 + [2.0 ** k] * 3 for k in range(L)], np.float32)
    rays = scenes.random_rays(200, rng, -1.5, 1.5)
    occ = _occupancy(L, R, rng)
    g = api.build_vdb(torch.from_numpy(occ).cuda(), boxes, ilog2)
    _check(g, occ, boxes, ilog2, rays, "build")
    # uint8 refresh: another structure, then one empty grid, then back
    other = _occupancy(L, R, rng)
    for k, state in enumerate((other, np.zeros_like(occ), np.ones_like(occ), occ)):
        g.refresh(torch.from_numpy(state).cuda())
        _check(g, state, boxes, ilog2, rays, f"refresh {k}")
    # density refreshes from the cache's side: the threshold is 0.5
    cache = torch.from_numpy(occ.astype(np.float32)).cuda()
    changed = torch.full((2,), -1, dtype=torch.int32, device="cuda")
    g.refresh_density(cache, None, threshold=0.5, changed=changed)
    assert changed.tolist() == [0, 0]
    _check(g, occ, boxes, ilog2, rays, "density, nothing")
    # one voxel of a mixed block flips: leaf bits only
    n = (R + 7) // 8
    pad = np.zeros((L,) + (8 * n,) * 3, np.uint8)
    pad[:, :R, :R, :R] = occ
    sums = pad.reshape(L, n, 8, n, 8, n, 8).sum((2, 4, 6))
    inner = np.argwhere((sums >= 2) & (sums <= 400))
    if len(inner):
        l, x, y, z = inner[rng.integers(0, len(inner))]
        at = np.argwhere(occ[l, 8 * x:8 * x + 8, 8 * y:8 * y + 8, 8 * z:8 * z + 8])[0] + 8 * np.asarray([x, y, z])
        state = occ.copy()
        state[l, at[0], at[1], at[2]] = 0
        dens = torch.from_numpy(state.astype(np.float32)).cuda()
        g.refresh_density(cache, dens, decay=0.25, threshold=0.5, changed=changed)
        assert changed.tolist() == [1, 0]
        np.testing.assert_array_equal(cache.cpu().numpy(), np.maximum(0.25 * occ, state).astype(np.float32))
        _check(g, state, boxes, ilog2, rays, "density, one voxel")
        occ = state
    # another structure
    dens = torch.from_numpy(other.astype(np.float32)).cuda()
    g.refresh_density(cache, dens, decay=0.25, threshold=0.5, changed=changed)
    flips = int((occ != other).sum())
    assert changed[0].item() == flips and (changed[1].item() == 1) == (flips > 0)
    _check(g, other, boxes, ilog2, rays, "density, restructured")
