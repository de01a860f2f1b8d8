"""The cursors' relocation and start estimates where they are least certain:
boxes far from the origin or of extreme size (the estimates' slack grows with
the coordinates over the voxel size), grids whose side is no multiple of a
block, small nodes (so whole root tiles are crossed), cells of every size next
to each other, and rays along planes.  Samples bit for bit against the
oracle's brute-force-pinned dense march."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api, scenes
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


# ------------------------------------------------------------------ rays walked in parts

def _parts_scene(levels, rng):
    R = 32
    occ = (rng.random((levels, R, R, R)) < 0.2).astype(np.uint8)
    boxes = np.asarray([[-(2.0 ** k)] * 3 + [2.0 ** k] * 3 for k in range(levels)], np.float32)
    step = {"kind": "const", "dt": 0.02, "cone": 0.0, "dt_min": 0.0} if levels == 1 else \
        {"kind": "cone", "dt": 0.0, "cone": 1.0 / 64.0, "dt_min": 0.02}
    return occ, boxes, step


@pytest.mark.parametrize("levels", [1, 3])
@pytest.mark.parametrize("n", [1, 63, 8193, 16384, 16385, 32769, 131073, 262144, 262145])
def test_ray_counts_around_the_part_numbers(n, levels):
    """Calls on both sides of every change of the number of parts, one-call
    (with short capacity too), two-phase, and walk and scan apart."""
    rng = np.random.default_rng(9200 + levels)
    occ, boxes, step = _parts_scene(levels, rng)
    o, d = scenes.random_rays(n, rng, -3.0, 3.0)
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.25, 6.0, step, "dense_branch")
    total = int(ref["offsets"][-1])
    od, dd = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
    for kind in ("vdb", "dist"):
        g = gpu_grid(kind, occ, boxes, 2)
        assert_same(gpu_sample(g, o, d, 0.25, 6.0, step, "branch", voxel_ids=False), ref, f"{kind} two-phase")
        for width, cap in ((0, total), (67, max(total - 5, 0))):
            s = api.Sampler(g, n, 0.25, 6.0, step, "branch", image_width=width)
            out = {"ray_ids": torch.full((cap,), -1, dtype=torch.int32, device="cuda"),
                   "t0": torch.zeros(cap, device="cuda"), "t1": torch.zeros(cap, device="cuda")}
            offsets, overflow = s.rays(od, dd, out["ray_ids"], out["t0"], out["t1"])
            got = {k: v.cpu().numpy() for k, v in out.items()}
            got["offsets"] = offsets.cpu().numpy()
            short = {k: v[:cap] if k != "offsets" else v for k, v in ref.items()}
            assert_same(got, short, f"{kind} width {width}")
            assert int(overflow.item()) == (1 if total > cap else 0)
        s.count_raw(od, dd)
        np.testing.assert_array_equal(s.scan().cpu().numpy(), ref["offsets"])


@pytest.mark.parametrize("n", [300, 40000])
def test_lost_runs_of_parts(n):
    """A voxel checkerboard gives every part more runs than its slots, and all
    of them more than the pool: lost parts are re-walked, their parts only."""
    R = 256
    i = np.arange(R)
    occ = ((i[:, None, None] + i[None, :, None] + i[None, None, :]) & 1).astype(np.uint8)[None]
    boxes = np.asarray([[-1, -1, -1, 1, 1, 1]], np.float32)
    rng = np.random.default_rng(9300)
    o = np.tile(np.asarray([[-3.0, 0.1, 0.2]], np.float32), (n, 1))
    aim = rng.uniform(-0.9, 0.9, (n, 3))
    d = aim - o
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    step = {"kind": "const", "dt": 0.004, "cone": 0.0, "dt_min": 0.0}
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.0, 8.0, step, "dense_branch")
    for kind, variant in (("vdb", "branch"), ("dense", "branch"), ("vdb", "skip")):
        got = gpu_sample(gpu_grid(kind, occ, boxes, 3), o, d, 0.0, 8.0, step, variant, voxel_ids=False)
        assert_same(got, ref, f"{kind} {variant}")
