"""Chunks of rows that many scenes share: scenes of a few rays, constant and
growing steps next to each other, scenes without rays and scenes whose range is
empty (far < near), which with a growing step have no table of points.  Scene
by scene bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api, scenes
from tests.test_gpu_batch import _run, _split
from tests.test_gpu_sampler import assert_same, gpu_grid

pytestmark = pytest.mark.gpu

CONST = {"kind": "const", "dt": 0.02, "cone": 0.0, "dt_min": 0.0}
CONE = {"kind": "cone", "dt": 0.0, "cone": 1 / 64, "dt_min": 0.01}


@pytest.mark.parametrize("variant", ["branch", "skip"])
@pytest.mark.parametrize("layout", ["tiny", "empty_ranges", "long_table", "uneven"])
def test_scenes_that_share_chunks(layout, variant):
    rng = np.random.default_rng(9890)
    occ = (rng.random((1, 24, 24, 24)) < 0.3).astype(np.uint8)
    boxes = np.asarray([[-1, -1, -1, 1, 1, 1]], np.float32)
    fine = {"kind": "cone", "dt": 0.0, "cone": 0.0, "dt_min": 6.0 / 9000}    # a table of 9,000 points
    plan = {"tiny": [(1 + s % 7, 0.25, 6.0, CONST if s % 3 else CONE) for s in range(64)],
            "empty_ranges": [(60, 0.25, 6.0, CONST), (50, 3.0, 2.0, CONE), (0, 0.25, 6.0, CONE), (40, 0.25, 6.0, CONE),
                             (30, 3.0, 2.0, CONST), (90, 0.0, 5.0, CONST), (20, 3.0, 2.0, CONE), (300, 0.25, 6.0, CONST)],
            "long_table": [(100, 0.0, 6.0, fine), (100, 0.25, 6.0, CONST), (400, 0.0, 6.0, fine)],
            "uneven": [(255, 0.25, 6.0, CONST), (2, 0.3, 5.0, CONE), (700, 0.25, 6.0, CONST), (1, 0.1, 4.0, CONE)]}[layout]
    g = gpu_grid("vdb", occ, boxes, 1)
    rays = [scenes.random_rays(n, rng, -2.0, 2.0) for n, *_ in plan]
    batch = api.Batch([(g, torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), near, far, step, 0)
                       for (o, d), (n, near, far, step) in zip(rays, plan)], variant, tune=(256, 2))
    res, _ = _run(batch)
    base = batch.info()["ray_base"]
    scene = oracle.Scene(occ, boxes)
    for s, ((o, d), (n, near, far, step)) in enumerate(zip(rays, plan)):
        ref = oracle.sample_rays(scene, o, d, near, far, step, "dense_branch")
        ref.pop("voxel_ids")
        assert_same(_split(res, base, n, s), ref, f"scene {s}")
