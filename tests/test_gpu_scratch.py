"""Calls that walk their rays in parts ask for more workspace; the calls that
the fixed scratch array held before still run on it, with as many parts as it
has room for, and a one-call pass runs on any workspace that holds whole rays.
Bit for bit against the call with the full workspace."""
import numpy as np
import pytest
import torch

from paper_2404_10272_amd import api, scenes
from tests.test_gpu_sampler import gpu_grid

pytestmark = pytest.mark.gpu

NEAR, FAR = 0.25, 6.0
STEP = {"kind": "const", "dt": 0.02, "cone": 0.0, "dt_min": 0.0}


def _case(n):
    rng = np.random.default_rng(9700)
    occ = (rng.random((1, 32, 32, 32)) < 0.2).astype(np.uint8)
    boxes = np.asarray([[-1, -1, -1, 1, 1, 1]], np.float32)
    o, d = scenes.random_rays(n, rng, -2.0, 2.0)
    return gpu_grid("vdb", occ, boxes, 2), torch.from_numpy(o).cuda(), torch.from_numpy(d).cuda()


def _out(n, cap):
    return (torch.full((cap,), -7, dtype=torch.int32, device="cuda"), torch.zeros(cap, device="cuda"),
            torch.zeros(cap, device="cuda"))


def _reference(g, o, d, sampler):
    offsets, _ = sampler.rays(o, d, *_out(0, 0))
    cap = int(offsets[-1].item())
    out = _out(0, cap)
    offsets, overflow = sampler.rays(o, d, *out)
    assert int(overflow.item()) == 0
    return cap, (offsets.clone(), *out)


@pytest.mark.parametrize("n", [16384, 98305, 131072, 200000, 262144, 300000])
def test_fixed_scratch_holds_every_call_of_up_to_440000_rays(n):
    g, o, d = _case(n)
    cap, ref = _reference(g, o, d, api.Sampler(g, n, NEAR, FAR, STEP, "branch"))
    offsets = torch.full((n + 1,), -3, dtype=torch.int64, device="cuda")
    overflow = torch.full((1,), 9, dtype=torch.int32, device="cuda")
    out = _out(n, cap)
    api.sample_rays_noalloc(g, o, d, NEAR, FAR, STEP, offsets, *out, overflow, "branch")
    torch.cuda.synchronize()
    for a, b in zip((offsets, *out), ref):
        assert torch.equal(a, b)
    assert int(overflow.item()) == 0


@pytest.mark.parametrize("n", [300, 20000, 131072])
def test_one_call_runs_on_less_workspace(n):
    g, o, d = _case(n)
    s = api.Sampler(g, n, NEAR, FAR, STEP, "branch")
    cap, ref = _reference(g, o, d, s)
    full = s.ws
    whole = 152 * n + 152 * 256 + 65536   # whole rays, and the pool's smallest size
    for size in (full.numel() - 256, full.numel() // 2, whole):
        if size < whole:
            continue
        s.ws, s.ws_bytes = full[:size], size
        out = _out(n, cap)
        offsets, overflow = s.rays(o, d, *out)
        torch.cuda.synchronize()
        for a, b in zip((offsets, *out), ref):
            assert torch.equal(a, b), size
    s.ws, s.ws_bytes = full[:100 * n], 100 * n
    with pytest.raises(api.OgvError):
        s.rays(o, d, *_out(n, cap))
