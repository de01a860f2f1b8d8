"""A part of a ray that has to be walked again, because the run pool had no
room for it, is cut at the parameters it was counted with: lattice points put
exactly on the cuts of one-level rays are written once, in their place."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api
from tests.test_gpu_sampler import gpu_grid

pytestmark = pytest.mark.gpu

R, HALF = 250, 1.5


def _ray_with_points_on_cuts(occ, boxes, rng):
    """A ray of the checkerboard and a step whose lattice has a point on the
    cut between two of its 16 parts, at which length * (j / 16) and the same
    by way of lengths over the voxel size round apart, in an occupied voxel."""
    f = np.float32
    scene = oracle.Scene(occ, boxes)
    inv_h = f(1) / ((f(HALF) + f(HALF)) / f(R))
    while True:
        o = np.asarray([-3.0, -2.9, -3.1], f) + rng.uniform(-0.05, 0.05, 3).astype(f)
        d = rng.uniform(0.9, 1.1, 3).astype(f)
        T = [oracle.planes(boxes[0], R, a, float(o[a]), float(d[a]))[1] for a in range(3)]
        E, X = max(t[0] for t in T), min(t[R] for t in T)
        length = X - E
        for j in range(1, 16):
            even = E + length * (f(j) * f(1 / 16))
            each = length * inv_h / f(16)
            other = E + length * ((f(j) * each) / (length * inv_h))
            if even == other:
                continue
            point = max(even, other)
            step = {"kind": "const", "dt": float(point / f(512)), "cone": 0.0, "dt_min": 0.0}
            ref = oracle.sample_rays(scene, o[None], d[None], 0.0, 8.0, step, "dense_branch")
            if point in ref["t0"]:
                return o, d, step, ref


@pytest.mark.parametrize("kind,variant", [("vdb", "branch"), ("dense", "branch"), ("vdb", "skip"), ("dist", "branch")])
def test_lost_parts_keep_their_cuts(kind, variant):
    rng = np.random.default_rng(9830)
    i = np.arange(R)
    occ = ((i[:, None, None] + i[None, :, None] + i[None, None, :]) & 1).astype(np.uint8)[None]
    boxes = np.asarray([[-HALF] * 3 + [HALF] * 3], np.float32)
    g = gpu_grid(kind, occ, boxes, 3)
    n = 600
    for _ in range(6):
        o, d, step, ref = _ray_with_points_on_cuts(occ, boxes, rng)
        s = api.Sampler(g, n, 0.0, 8.0, step, variant)
        per = ref["t0"].size
        ids = torch.full((n * per,), -1, dtype=torch.int32, device="cuda")
        t0 = torch.full((n * per,), -1.0, device="cuda")
        t1 = torch.full((n * per,), -1.0, device="cuda")
        od = torch.from_numpy(np.tile(o, (n, 1))).cuda()
        dd = torch.from_numpy(np.tile(d, (n, 1))).cuda()
        offsets, overflow = s.rays(od, dd, ids, t0, t1)
        np.testing.assert_array_equal(offsets.cpu().numpy(), per * np.arange(n + 1))
        assert int(overflow.item()) == 0
        np.testing.assert_array_equal(t0.cpu().numpy().reshape(n, per), np.tile(ref["t0"], (n, 1)))
        np.testing.assert_array_equal(t1.cpu().numpy().reshape(n, per), np.tile(ref["t1"], (n, 1)))
        np.testing.assert_array_equal(ids.cpu().numpy(), np.repeat(np.arange(n), per))
        s.count(od, dd)
        t0.fill_(-1.0)
        s.fill(od, dd, ids, t0, t1)
        np.testing.assert_array_equal(t0.cpu().numpy().reshape(n, per), np.tile(ref["t0"], (n, 1)))
