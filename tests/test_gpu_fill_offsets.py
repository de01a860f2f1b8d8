"""The emission pass writes where its offsets say: offsets of a count, moved by
a constant (a program that packs several calls into one set of arrays), at ray
counts that are walked in parts and whole, with lost runs and without."""
import numpy as np
import pytest
import torch

import oracle
from paper_2404_10272_amd import api, scenes
from tests.test_gpu_sampler import gpu_grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,board", [(n, False) for n in (1, 300, 20000, 40001, 262145)] +
                         [(n, True) for n in (1, 300, 20000, 40001)])
def test_offsets_moved_by_a_constant(n, board):
    rng = np.random.default_rng(9840)
    R, step = 32, {"kind": "const", "dt": 0.02, "cone": 0.0, "dt_min": 0.0}
    occ = (rng.random((1, R, R, R)) < 0.2).astype(np.uint8)
    if board:      # more runs than the pool holds
        R = 256
        i = np.arange(R)
        occ = ((i[:, None, None] + i[None, :, None] + i[None, None, :]) & 1).astype(np.uint8)[None]
    boxes = np.asarray([[-1, -1, -1, 1, 1, 1]], np.float32)
    o, d = scenes.random_rays(n, rng, -2.0, 2.0)
    ref = oracle.sample_rays(oracle.Scene(occ, boxes), o, d, 0.25, 6.0, step, "dense_branch")
    total = int(ref["offsets"][-1])
    od, dd = torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()
    s = api.Sampler(gpu_grid("vdb", occ, boxes, 2), n, 0.25, 6.0, step, "branch")
    for shift, spare in ((3, 5), (1000, 0), (8, -2)):
        s.count(od, dd)
        s.offsets += shift
        cap = max(total + shift + spare, 0)
        ids = torch.full((cap,), -9, dtype=torch.int32, device="cuda")
        t0 = torch.full((cap,), -9.0, device="cuda")
        t1 = torch.full((cap,), -9.0, device="cuda")
        s.fill(od, dd, ids, t0, t1)
        for got, key in ((ids, "ray_ids"), (t0, "t0"), (t1, "t1")):
            got = got.cpu().numpy()
            want = np.full(cap, -9, got.dtype)
            want[shift:shift + total] = ref[key][:max(cap - shift, 0)]
            np.testing.assert_array_equal(got, want, err_msg=f"{key} {shift} {spare}")
