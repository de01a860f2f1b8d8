"""The expansion at the edges of its choices: growing-step lattices on both
sides of the size kept in LDS, runs of one to a few samples (a 16-byte group
of outputs holds up to four runs), arrays with no 16-byte alignment, and
chunks of rows that several scenes share.  Bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api, scenes
from tests.test_gpu_batch import _run, _split
from tests.test_gpu_sampler import assert_same, gpu_grid, gpu_sample

pytestmark = pytest.mark.gpu

FAR = 3.0


def _scene(rng, R=64):
    occ = (rng.random((1, R, R, R)) < 0.35).astype(np.uint8)   # runs of one or two voxels, and longer
    return occ, np.asarray([[-1, -1, -1, 1, 1, 1]], np.float32)


def _cone(points):
    """A growing step whose table takes `points` entries at the most (18 of them to spare)."""
    return {"kind": "cone", "dt": 0.0, "cone": 0.0, "dt_min": FAR / (points - 18)}


@pytest.mark.parametrize("points", [40, 300, 4090, 4096, 4097, 4200])
@pytest.mark.parametrize("n", [257, 20000])
def test_growing_steps_around_the_table_in_lds(n, points):
    rng = np.random.default_rng(9400 + points)
    occ, boxes = _scene(rng)
    n = n if points < 4000 else min(n, 2000)
    o, d = scenes.random_rays(n, rng, -1.5, 1.5)
    step = _cone(points)
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.0, FAR, step, "dense_branch")
    for kind in ("vdb", "dense"):
        got = gpu_sample(gpu_grid(kind, occ, boxes, 2), o, d, 0.0, FAR, step, "branch", voxel_ids=False)
        assert_same(got, ref, f"{kind} two-phase")


@pytest.mark.parametrize("shift", [0, 1, 3])
@pytest.mark.parametrize("dt", [0.2, 0.03, 0.004])
def test_short_runs_and_unaligned_arrays(dt, shift):
    rng = np.random.default_rng(9500)
    occ, boxes = _scene(rng)
    n = 3000
    o, d = scenes.random_rays(n, rng, -1.5, 1.5)
    step = {"kind": "const", "dt": dt, "cone": 0.0, "dt_min": 0.0}
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.0, FAR, step, "dense_branch")
    total = int(ref["offsets"][-1])
    s = api.Sampler(gpu_grid("vdb", occ, boxes, 2), n, 0.0, FAR, step, "branch")
    cap = total - 3
    out = {"ray_ids": torch.full((cap + shift + 1,), -7, dtype=torch.int32, device="cuda"),
           "t0": torch.full((cap + shift + 1,), -7.0, device="cuda"), "t1": torch.full((cap + shift + 1,), -7.0, device="cuda")}
    offsets, overflow = s.rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(),
                               *(out[k][shift:shift + cap] for k in ("ray_ids", "t0", "t1")))
    got = {k: v[shift:shift + cap].cpu().numpy() for k, v in out.items()}
    got["offsets"] = offsets.cpu().numpy()
    assert_same(got, {k: v[:cap] if k != "offsets" else v for k, v in ref.items()}, "short")
    assert int(overflow.item()) == 1
    for k, v in out.items():   # nothing beside the arrays is written
        assert (v[:shift].cpu().numpy() == -7).all() and (v[shift + cap:].cpu().numpy() == -7).all(), k


@pytest.mark.parametrize("counts", [(5, 1, 70, 300, 256, 2, 900), (1, 255, 1, 255, 512), (3000, 40)])
def test_scenes_sharing_chunks(counts):
    rng = np.random.default_rng(9600 + len(counts))
    gs, refs = [], []
    for i, n in enumerate(counts):
        occ, boxes = _scene(rng, 32)
        o, d = scenes.random_rays(n, rng, -1.5, 1.5)
        step = _cone(200 + i) if i % 3 == 1 else {"kind": "const", "dt": 0.01 * (1 + i), "cone": 0.0, "dt_min": 0.0}
        refs.append(oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.0, FAR, step, "dense_branch"))
        gs.append((api.build_vdb(torch.from_numpy(occ).cuda(), boxes, 2), torch.from_numpy(o).cuda(),
                   torch.from_numpy(d).cuda(), 0.0, FAR, step, 0))
    batch = api.Batch(gs, "branch")
    res, _ = _run(batch)
    base = batch.info()["ray_base"]
    for s, n in enumerate(counts):
        got = _split(res, base, n, s)
        for k in ("offsets", "ray_ids", "t0", "t1"):
            np.testing.assert_array_equal(got[k], refs[s][k], err_msg=f"scene {s} {k}")
