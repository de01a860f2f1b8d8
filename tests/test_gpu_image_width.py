"""An image far wider than the call has rays: the option changes speed alone."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api, scenes
from tests.test_gpu_batch import _run, _split
from tests.test_gpu_sampler import assert_same, gpu_grid, gpu_sample

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 7, 1000])
@pytest.mark.parametrize("width", [1000, 1001, 5000, 1 << 22, 1 << 27])
def test_images_wider_than_the_rays(n, width):
    rng = np.random.default_rng(9880)
    for levels in (1, 2):
        occ = (rng.random((levels, 16, 16, 16)) < 0.3).astype(np.uint8)
        boxes = np.asarray([[-(2.0 ** k)] * 3 + [2.0 ** k] * 3 for k in range(levels)], np.float32)
        o, d = scenes.random_rays(n, rng, -2.0, 2.0)
        step = {"kind": "const", "dt": 0.02, "cone": 0.0, "dt_min": 0.0}
        ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.25, 6.0, step, "dense_branch")
        g = gpu_grid("vdb", occ, boxes, 1)
        got = gpu_sample(g, o, d, 0.25, 6.0, step, "branch", voxel_ids=False, image_width=width)
        assert_same(got, ref, f"{levels} levels")


def test_batch_of_images_wider_than_their_rays():
    rng = np.random.default_rng(9881)
    occ = (rng.random((1, 16, 16, 16)) < 0.3).astype(np.uint8)
    boxes = np.asarray([[-1, -1, -1, 1, 1, 1]], np.float32)
    step = {"kind": "const", "dt": 0.02, "cone": 0.0, "dt_min": 0.0}
    g = gpu_grid("vdb", occ, boxes, 1)
    rays = [scenes.random_rays(n, rng, -2.0, 2.0) for n in (5, 700, 64)]
    batch = api.Batch([(g, torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), 0.25, 6.0, step, w)
                       for (o, d), w in zip(rays, (3000, 701, 64))], "branch", tune=(256, 2))
    res, _ = _run(batch)
    base = batch.info()["ray_base"]
    for s, (o, d) in enumerate(rays):
        ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.25, 6.0, step, "dense_branch")
        ref.pop("voxel_ids")
        assert_same(_split(res, base, o.shape[0], s), ref, f"scene {s}")
