"""A workspace sized for one ray count serves every smaller one, in each form
of the call."""
import numpy as np
import pytest
import torch

from paper_2404_10272_amd import api
from tests.test_gpu_scratch import FAR, NEAR, STEP, _case, _out, _reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,size_for", [(200000, 300000), (131072, 200000), (262144, 262145), (16384, 17000), (300, 524289)])
def test_count_and_fill_on_the_workspace_of_more_rays(n, size_for):
    g, o, d = _case(n)
    s = api.Sampler(g, n, NEAR, FAR, STEP, "branch")
    cap, ref = _reference(g, o, d, s)
    big = api.workspace_bytes(size_for, NEAR, FAR, s.step)
    s.ws, s.ws_bytes = torch.empty(big, dtype=torch.uint8, device="cuda"), big
    for raw in (False, True):
        if raw:
            s.count_raw(o, d)
            s.scan()
        else:
            s.count(o, d)
        out = _out(n, cap)
        s.fill(o, d, *out)
        torch.cuda.synchronize()
        for a, b in zip((s.offsets, *out), ref):
            assert torch.equal(a, b)
