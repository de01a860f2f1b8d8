"""The cursors' relocation and start estimates where they are least certain:
boxes far from the origin or of extreme size (the estimates' slack grows with
the coordinates over the voxel size), grids whose side is no multiple of a
block, small nodes (so whole root tiles are crossed), cells of every size next
to each other, and rays along planes.  Samples bit for bit against the
oracle's brute-force-pinned dense march."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_sampler import VARIANTS, assert_same, gpu_grid, gpu_sample

pytestmark = pytest.mark.gpu

# side, node log2, box centre, box half width
GRIDS = [(40, 1, (0.0, 0.0, 0.0), 1.0), (72, 2, (1000.0, -500.0, 250.0), 0.5), (100, 3, (1.0, 1.0, -1.0), 1e-3),
         (64, 1, (-3e4, 7.0, 2e5), 1e4)]


def _blocks(rng, R):
    """Occupancy of 8^3 blocks: most empty, some full, some of full and empty
    4^3 quarters, some of random voxels; whole corners empty."""
    n = (R + 7) // 8
    occ = np.zeros((n * 8,) * 3, np.uint8)
    for b in np.ndindex(n, n, n):
        at = tuple(slice(8 * i, 8 * i + 8) for i in b)
        kind = rng.integers(0, 10)
        if kind == 0:
            occ[at] = 1
        elif kind == 1:
            occ[at] = np.kron(rng.integers(0, 2, (2, 2, 2)), np.ones((4, 4, 4))).astype(np.uint8)
        elif kind == 2:
            occ[at] = rng.random((8, 8, 8)) < 0.3
    half = n * 4 // 8 * 8
    occ[:half, :half, :] = 0
    return occ[:R, :R, :R][None]


def _rays(rng, centre, half, R, n):
    aim = centre + rng.uniform(-half, half, (n, 3))
    d = rng.normal(size=(n, 3))
    kind = rng.integers(0, 4, n)
    d[kind == 1, rng.integers(0, 3)] = 0.0                        # one axis still
    d[kind == 2] = np.round(d[kind == 2])                         # diagonals: crossings tie
    d[np.abs(d).sum(1) == 0] = 1.0
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    snap = kind == 3                                              # through lattice corners
    aim[snap] = centre - half + np.round((aim[snap] - centre + half) / (2 * half / R)) * (2 * half / R)
    o = aim - d * half * rng.uniform(0.0, 4.0, (n, 1))
    return o.astype(np.float32), d.astype(np.float32)


@pytest.mark.parametrize("grid", GRIDS, ids=lambda g: f"{g[0]}-{g[3]:g}")
def test_walks_where_estimates_are_uncertain(grid):
    R, ilog2, centre, half = grid
    rng = np.random.default_rng(9100 + R)
    occ = _blocks(rng, R)
    c = np.asarray(centre, np.float64)
    boxes = np.concatenate([c - half, c + half]).astype(np.float32)[None]
    o, d = _rays(rng, c, half, R, 2000)
    near, far = 0.0, float(np.float32(8.0 * half))
    step = {"kind": "const", "dt": float(np.float32(half / 150.0)), "cone": 0.0, "dt_min": 0.0}
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, near, far, step, "dense_branch", ilog2=ilog2)
    assert ref["offsets"][-1] > 10000
    for kind, variant in VARIANTS:
        got = gpu_sample(gpu_grid(kind, occ, boxes, ilog2), o, d, near, far, step, variant, voxel_ids=False)
        assert_same(got, ref, f"{kind} {variant}")
