"""The ray walk's own code compiled for the host: rays walked in parts against
the same rays walked whole, and relocations of rays with still axes, on the CPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("walk") / "walk_host.so")
    subprocess.run(["hipcc", "--offload-host-only", "-std=c++17", "-O1", "-fPIC", "-shared", "-ffp-contract=off", "-w",
                    os.path.join(HERE, "walk_host.hip"), "-o", so], check=True)
    return ctypes.CDLL(so)


class Grid:
    def __init__(self, occ, boxes):
        occ = np.asarray(occ, np.uint8)
        boxes = np.asarray(boxes, np.float32)
        self.L, self.R = occ.shape[:2]
        self.bits = np.packbits(occ.reshape(-1) != 0, bitorder="little")
        self.bits = np.concatenate([self.bits, np.zeros(-len(self.bits) % 4, np.uint8)]).view(np.uint32)
        self.geom = np.zeros((self.L, 12), np.float32)
        self.geom[:, :3] = boxes[:, :3]
        self.geom[:, 3:6] = (boxes[:, 3:] - boxes[:, :3]) / np.float32(self.R)
        self.geom[:, 6:9] = np.float32(1) / self.geom[:, 3:6]


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def runs_of(walk, g, o, d, near, far, part=(0, 1), single=False, cap=4096):
    out = np.zeros((cap, 2), np.float32)
    n = walk.walk_runs(g.L, g.R, _p(g.geom), _p(g.bits), _p(o), _p(d), ctypes.c_float(near), ctypes.c_float(far),
                       part[0], part[1], int(single), _p(out), cap)
    assert n <= cap
    return out[:n]


def covered(runs):
    """Runs as maximal intervals, the empty ones left out."""
    out = []
    for lo, hi in runs:
        if not lo < hi:
            continue
        if out and out[-1][1] == lo:
            out[-1][1] = hi
        else:
            out.append([lo, hi])
    return out


def in_parts(walk, g, o, d, near, far, n, single=False):
    return np.concatenate([runs_of(walk, g, o, d, near, far, (j, n), single) for j in range(n)])


def _cascades(levels, R, rng, fill):
    occ = (rng.random((levels, R, R, R)) < fill).astype(np.uint8)
    return Grid(occ, [[-1.5 * 2.0 ** k] * 3 + [1.5 * 2.0 ** k] * 3 for k in range(levels)])


def _same_inside(whole, parts, near, far, what):
    """The same parameters of [near, far] covered, each once."""
    def clip(iv):
        return [[max(lo, np.nextafter(np.float32(near), np.float32(-np.inf))), min(hi, np.float32(far))]
                for lo, hi in iv if hi >= near and lo < far]
    assert covered(clip(covered(whole))) == covered(clip(covered(parts))), what
    length = lambda iv: sum(float(hi) - float(lo) for lo, hi in clip([r for r in iv if r[0] < r[1]]))
    assert abs(length(whole) - length(parts)) <= 1e-5 * (1.0 + length(whole)), what


@pytest.mark.parametrize("parts", [2, 4, 8, 16])
@pytest.mark.parametrize("levels", [2, 3, 4])
def test_parts_of_a_range_of_no_length(walk, levels, parts):
    """near == far, and rays that leave the outermost box exactly at near: the
    range holds one parameter, which one part owns."""
    rng = np.random.default_rng(9800 + levels)
    g = _cascades(levels, 16, rng, 1.1)
    edge = np.float32(1.5 * 2.0 ** (levels - 1))
    for k in range(30):
        o = rng.uniform(-1.0, 1.0, 3).astype(np.float32)
        d = rng.normal(size=3).astype(np.float32)
        near = np.float32(rng.uniform(0.0, 1.0))
        far = near
        if k % 3 == 0:      # out through a face at t = 0
            o[0], d[0] = edge, abs(d[0]) + np.float32(0.1)
            near, far = np.float32(0), np.float32(2)
        whole = runs_of(walk, g, o, d, near, far)
        assert any(lo < near <= hi for lo, hi in whole)
        got = in_parts(walk, g, o, d, near, far, parts)
        assert sum(bool(lo < near <= hi) for lo, hi in got) == 1, (k, got)


@pytest.mark.parametrize("parts", [2, 4, 16])
def test_parts_cover_a_cascade_ray_once(walk, parts):
    rng = np.random.default_rng(9810)
    g = _cascades(3, 24, rng, 0.4)
    for k in range(300):
        o = rng.uniform(-4.0, 4.0, 3).astype(np.float32)
        d = (rng.uniform(-3.0, 3.0, 3) - o).astype(np.float32)
        if k % 4 == 0:      # grazes the inner box: a segment of almost no length in the middle of the ray
            o = np.asarray([-4.0, 1.5 - 3e-7 * (k % 7), 0.1], np.float32)
            d = np.asarray([1.0, 0.0, 0.0], np.float32)
        near, far = np.float32(0.1 * (k % 3)), np.float32([3.0, 9.0, 100.0][k % 3])
        _same_inside(runs_of(walk, g, o, d, near, far), in_parts(walk, g, o, d, near, far, parts), near, far, k)


@pytest.mark.parametrize("R", [100, 128, 250])
def test_both_walks_cut_a_one_level_ray_alike(walk, R):
    """A part counted by the walk of one-level grids is walked again, when its
    runs were lost, by the walk of any number of levels."""
    rng = np.random.default_rng(9835)
    g = Grid(np.ones((1, R, R, R)), [[-1.5] * 3 + [1.5] * 3])
    for k in range(100):
        o = rng.uniform(-4.0, 4.0, 3).astype(np.float32)
        d = (rng.uniform(-1.4, 1.4, 3) - o).astype(np.float32)
        n = 2 ** int(rng.integers(1, 5))
        near, far = [(0.0, 8.0), (0.4, 0.9), (0.5, 0.5)][k % 3]
        for j in range(n):
            # runs behind far hold no samples, and either walk may leave them out
            one, any_level = ([tuple(r) for r in runs_of(walk, g, o, d, near, far, (j, n), single) if r[0] < far]
                              for single in (True, False))
            assert one == any_level, (k, j, n)


@pytest.mark.parametrize("still", [[], [0], [2], [0, 1], [1, 2]])
def test_still_axes_leave_relocations_to_the_estimate(walk, still):
    """A ray along grid planes settles as many relocations by the estimate as any
    other: its still axes keep their voxels."""
    rng = np.random.default_rng(9840)
    R = 128
    g = Grid(np.ones((1, 8, 8, 8)), [[-1.5] * 3 + [1.5] * 3])
    g.geom[0, 3:6] = np.float32(3) / np.float32(R)
    g.geom[0, 6:9] = np.float32(1) / g.geom[0, 3:6]
    h = float(g.geom[0, 3])
    exact = 0
    for k in range(400):
        o = rng.uniform(-1.4, 1.4, 3).astype(np.float32)
        d = rng.uniform(0.2, 1.0, 3).astype(np.float32)
        d[still] = 0.0
        w = np.floor((o.astype(np.float64) + 1.5) / h).astype(np.int32) & ~7    # its 8^3 block, entered somewhere
        p = (w + 8).astype(np.int32)
        at = np.floor((o.astype(np.float64) + 1.5) / h).astype(np.int32)
        moving = [a for a in range(3) if a not in still]
        t = np.float32(min((-1.5 + float(p[a]) * h - float(o[a])) / float(d[a]) for a in moving) * rng.uniform(0.05, 0.95))
        got = w.copy()
        got[still] = at[still]
        exact += walk.relocation(R, _p(g.geom), _p(o), _p(d), _p(got), _p(p), ctypes.c_float(t)) > 0
        want = np.floor((o + d.astype(np.float64) * float(t) + 1.5) / h).astype(np.int32)
        want[still] = at[still]
        assert (np.abs(got - want) <= 0).all() or np.abs((o + d.astype(np.float64) * float(t) + 1.5) / h % 1 - 0.5).max() > 0.4999
    assert exact <= 8, exact
