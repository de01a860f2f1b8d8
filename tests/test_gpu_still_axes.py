"""Rays along grid axes and planes, whose still axes are never crossed: on boxes
from tiny to huge, with ranges up to the largest float, through every cursor.
Samples bit for bit against the oracle."""
import numpy as np
import pytest

import oracle
from tests.test_gpu_sampler import VARIANTS, assert_same, gpu_grid, gpu_sample
from tests.test_gpu_walk import _blocks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("half,centre,speed", [(1.0, 0.0, 1.0), (1e-3, 5.0, 1.0), (1e4, -3e5, 1.0), (1.0, 0.0, 1e-38),
                                               (1.0, 0.25, 6e-39), (1e31, 0.0, 1.0), (1e31, 3e31, 1e-3)])
@pytest.mark.parametrize("levels", [1, 2])
def test_rays_along_axes_and_planes(levels, half, centre, speed):
    rng = np.random.default_rng(9920)
    R, n = 72, 1500
    occ = np.concatenate([_blocks(rng, R) for _ in range(levels)])
    boxes = np.asarray([[centre - half * 2.0 ** k] * 3 + [centre + half * 2.0 ** k] * 3 for k in range(levels)], np.float32)
    outer = half * 2.0 ** (levels - 1)
    d = rng.normal(size=(n, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    still = rng.integers(0, 3, n)
    d[np.arange(n), still] = 0.0
    two = rng.random(n) < 0.5
    d[np.arange(n)[two], (still[two] + 1) % 3] = 0.0
    d[:7] = 0.0                                                # and none moving at all
    o = centre + rng.uniform(-outer, outer, (n, 3)) - d * outer * rng.uniform(0.0, 1.5, (n, 1))
    far = np.float32(min(4.0 * outer / speed, 3.4e38))
    step = {"kind": "const", "dt": float(np.float32(far / 3000.0)), "cone": 0.0, "dt_min": 0.0}
    o, d = o.astype(np.float32), (d * speed).astype(np.float32)
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.0, far, step, "dense_branch", ilog2=2)
    assert ref["offsets"][-1] > 10000
    for kind, variant in VARIANTS:
        got = gpu_sample(gpu_grid(kind, occ, boxes, 2), o, d, 0.0, far, step, variant, voxel_ids=False)
        assert_same(got, ref, f"{kind} {variant}")
