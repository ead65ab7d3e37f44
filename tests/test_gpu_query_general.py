"""The probe query at any point and on any texels a caller has: points beyond
every bound use the volume's outermost probes, and a texel that is no finite
number shows wherever the oracle's blend shows it."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as o
from paper_2108_05263_amd import scenegen as sg

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def _volume(dims, texel="f32"):
    cfg = dataclasses.replace(sg.CONFIGS["hd"], probe_dims=dims, probe_spacing=2.0, probe_texel=texel)
    return sg.make_probe_grid(cfg)


def _query(grid, irr, dep, p, n):
    from paper_2108_05263_amd import gi
    pr = gi.Probes(grid)
    pr.load(irr, dep)
    return gi.probe_query(pr, torch.from_numpy(p).cuda(), torch.from_numpy(n).cuda()).cpu().numpy()


@pytest.mark.parametrize("texel", ["f32", "f16"])
@pytest.mark.parametrize("far", [1e20, 1e38, 3.4e38, np.inf])
def test_far_points_take_the_outermost_probes(far, texel):
    dims = (5, 3, 4)
    grid = _volume(dims, texel)
    irr, dep = sg.random_probe_textures(grid, 3)
    i = np.arange(grid.count)
    place = np.stack([i % dims[0], i // dims[0] % dims[1], i // (dims[0] * dims[1])], 1).astype(np.float32)
    irr[..., :3] = place[:, None]             # every probe holds its own index
    centre = np.asarray(grid.lo) + np.asarray(grid.spacing) * (np.asarray(dims) * 0.5)
    p = np.tile(centre.astype(np.float32), (6, 1))
    for a in range(3):
        p[2 * a, a], p[2 * a + 1, a] = far, -far
    n = np.tile(np.float32([0, 0, 1]), (6, 1))
    q = _query(grid, irr, dep, p, n)
    for a in range(3):
        # a blend of equal values: the outermost index up to FP32 rounding
        assert abs(q[2 * a, a] - (dims[a] - 1)) < 1e-5 * dims[a] and abs(q[2 * a + 1, a]) < 1e-5


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_texels_of_weight_zero_show_as_in_the_oracle(axis, bad):
    grid = _volume((2, 2, 2))
    irr, dep = sg.random_probe_textures(grid, 3)
    irr[[0, 7]] = bad                          # two opposite corners of the one cell
    rng = np.random.default_rng(1)
    lo, hi = np.asarray(grid.lo), np.asarray(grid.lo) + np.asarray(grid.spacing) * 2
    p = rng.uniform(lo, hi, (64, 3)).astype(np.float32)
    p[:32, axis], p[32:, axis] = lo[axis] - 1, hi[axis] + 1       # the other layer has weight zero
    n = rng.normal(size=(64, 3))
    n = (n / np.linalg.norm(n, axis=1)[:, None]).astype(np.float32)
    q, ref = _query(grid, irr, dep, p, n), o.probe_query(grid, irr, dep, p, n)
    assert np.array_equal(np.isfinite(q), np.isfinite(ref))
