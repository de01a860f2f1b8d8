"""Cascade rays walked in parts whose range has no length, or a segment of
almost none: near == far, rays that leave the outermost box exactly at near,
rays along an inner box's face.  At ray counts on both sides of every number
of parts, bit for bit against the oracle, with voxel ids and without."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api
from tests.test_gpu_sampler import assert_same, gpu_grid, gpu_sample

pytestmark = pytest.mark.gpu


def _rays(case, levels, n, rng):
    edge = 2.0 ** (levels - 1)
    o = rng.uniform(-1.0, 1.0, (n, 3))
    d = rng.normal(size=(n, 3))
    near, far = 0.5, 0.5
    if case == "exit":          # through a face of the outermost box at t = 0
        a = rng.integers(0, 3, n)
        o[np.arange(n), a] = edge
        d[np.arange(n), a] = np.abs(d[np.arange(n), a]) + 0.1
        near, far = 0.0, 3.0
    elif case == "graze":       # along the innermost box's face
        o[:, 0], o[:, 1] = -edge, 1.0 - 6e-8 * rng.integers(0, 5, n)
        d[:] = [1.0, 0.0, 0.0]
        near, far = 0.0, 8.0 * edge
    return o.astype(np.float32), d.astype(np.float32), near, far


@pytest.mark.parametrize("n", [1, 300, 20000, 100000, 262144, 262145])
@pytest.mark.parametrize("case", ["point", "exit", "graze"])
@pytest.mark.parametrize("levels", [2, 3, 4])
def test_ranges_and_segments_of_no_length(levels, case, n):
    rng = np.random.default_rng(9820 + levels)
    R = 16
    occ = (rng.random((levels, R, R, R)) < 0.7).astype(np.uint8)
    boxes = np.asarray([[-(2.0 ** k)] * 3 + [2.0 ** k] * 3 for k in range(levels)], np.float32)
    o, d, near, far = _rays(case, levels, n, rng)
    step = {"kind": "const", "dt": 0.25, "cone": 0.0, "dt_min": 0.0}
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, near, far, step, "dense_branch")
    assert ref["offsets"][-1] > 0 or n == 1
    for kind in ("vdb", "dense"):
        g = gpu_grid(kind, occ, boxes, 1)
        for vox in (False, True):
            assert_same(gpu_sample(g, o, d, near, far, step, "branch", voxel_ids=vox), ref, f"{kind} {vox}")
        s = api.Sampler(g, n, near, far, step, "skip")
        total = int(ref["offsets"][-1])
        out = {"ray_ids": torch.full((total,), -1, dtype=torch.int32, device="cuda"),
               "t0": torch.zeros(total, device="cuda"), "t1": torch.zeros(total, device="cuda")}
        offsets, _ = s.rays(torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda(), out["ray_ids"], out["t0"], out["t1"])
        got = {k: v.cpu().numpy() for k, v in out.items()}
        got["offsets"] = offsets.cpu().numpy()
        assert_same(got, ref, f"{kind} one call")
