"""The staged pixel form of the initial pass on interleaved primitive types.

It reorders each staged cell's items (spheres, then boxes).  With the room's
primitives renumbered in a shuffled order the reordering swaps items in most
cells; the frames stay those of the walk over the caller's id-ordered lists,
bit for bit.  Few candidates, emitter candidates and middling image sizes are
what reaches that form; many candidates (the last case) take the tile form,
whose lists separate the types too.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2108_05263_amd import scenegen as sg
from test_gpu_parity import _lds_vs_global

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("room,W,H,M,M_light,texel", [
    ("hd", 250, 141, 4, 0, "f32"), ("hd", 333, 201, 5, 0, "f16"), ("hd", 250, 141, 8, 4, "f32"), ("hd", 640, 360, 13, 0, "f32"),
    ("glossy", 250, 141, 4, 3, "f16"), ("hd", 250, 141, 32, 0, "f32"),
])
def test_staged_cells_of_interleaved_types(room, W, H, M, M_light, texel):
    from paper_2108_05263_amd import gi
    cfg = sg.CONFIGS[room]
    cfg = dataclasses.replace(cfg, probe_dims=(8, 4, 8), probe_spacing=cfg.room_hi[0] / 8, probe_texel=texel,
                              params=dataclasses.replace(cfg.params, M=M, M_light=M_light))
    sc = sg.make_scene(cfg)
    sc = dataclasses.replace(sc, prims=np.ascontiguousarray(sc.prims[np.random.default_rng(5).permutation(sc.n_prims)]))
    types = sc.prims.view(np.uint32)[:, 3].astype(np.int64)
    assert np.sum(np.diff(types) != 0) > sc.n_prims // 4
    _lds_vs_global(gi, cfg, sc, *sg.random_probe_textures(sg.make_probe_grid(cfg), 3), W, H)
