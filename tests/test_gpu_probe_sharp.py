"""Depth texels of the probe update where the weights leave the normal range.

A sky that is no finite number makes the update take its rays one by one, with
a branch on the texel's side; the depth filter reads no radiance, so its
texels have to keep every bit.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2108_05263_amd import scenegen as sg

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("texel", ["f32", "f16"])
@pytest.mark.parametrize("rays", [64, 203])
@pytest.mark.parametrize("sharpness", [1.0, 50.0, 1e3, 1e4, 1e5])
def test_depth_texels_do_not_depend_on_the_radiance(sharpness, rays, texel):
    from paper_2108_05263_amd import gi
    cfg = dataclasses.replace(sg.CONFIGS["hd"], probe_dims=(4, 2, 4), probe_spacing=8.0, probe_texel=texel)
    scene, grid = sg.make_scene(cfg), sg.make_probe_grid(cfg)
    out = []
    for sky in (1.0, np.inf):
        ds = gi.DeviceScene(dataclasses.replace(scene, has_room=False, sky=np.full(3, sky, np.float32)), cfg.grid_res)
        a, b = gi.Probes(grid), gi.Probes(grid)
        a.load(*sg.random_probe_textures(grid, 3))
        gi.probe_update(ds, a, b, rays, 0.5, sharpness, 7, 3)
        torch.cuda.synchronize()
        out.append((b.irr.clone(), b.dep.clone()))
    assert torch.isfinite(out[0][0]).all() and not torch.isfinite(out[1][0]).all()
    assert torch.equal(out[0][1].view(torch.uint8), out[1][1].view(torch.uint8))
