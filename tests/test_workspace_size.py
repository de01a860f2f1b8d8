"""The workspace size a call reports never falls as its rays grow (no GPU)."""
import pytest

from paper_2404_10272_amd import api


@pytest.mark.parametrize("step", [dict(kind="const", dt=0.02), dict(kind="cone", cone=1 / 64, dt_min=0.02)])
def test_size_never_falls_as_rays_grow(step):
    st = api.make_step(step)
    counts = [0, 1, 255, 257, 8192, 16383, 16384, 16385, 20000, 32768, 32769, 65536, 100000, 131072, 131073, 200000,
              262143, 262144, 262145, 300000, 400000, 440000, 524288, 524289, 600000, 1000000]
    sizes = [api.workspace_bytes(n, 0.25, 6.0, st) for n in counts]
    assert sizes == sorted(sizes), list(zip(counts, sizes))
    assert max(s - 153 * n for n, s in zip(counts, sizes)) <= 81 << 20   # whole rays and 80 MB
