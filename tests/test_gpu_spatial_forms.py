"""The spatial pass's ways of reaching the scene: staged for 256 threads, staged
for the 768 threads of a 48x16 tile, and read from global memory (with the
grid or the brute-force loop).  Only where the walk reads differs, so every
output bit has to agree; the pass itself is checked against the oracle by
the parity tests.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2108_05263_amd import scenegen as sg

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def gi():
    from paper_2108_05263_amd import gi as g
    g.load()
    return g


# edges of both tile widths and of one pixel; no, some and the most
# neighbours; both normalisations and G-buffer formats; an open scene
@pytest.mark.parametrize("room,W,H,kw", [
    ("hd", 16, 16, {}), ("hd", 17, 33, {"k": 8}), ("hd", 250, 141, {"k": 0}), ("hd", 1, 1, {}),
    ("uhd", 48, 16, {}), ("uhd", 49, 17, {"k": 8}), ("uhd", 385, 217, {}), ("uhd", 95, 31, {"unbiased": 0}),
    ("uhd", 200, 100, {"open": True}), ("glossy", 101, 67, {"k": 8}), ("hd", 333, 50, {"gb_format": "f16"}),
])
def test_spatial_scene_access_is_bit_identical(gi, room, W, H, kw):
    kw = dict(kw)
    gbf, open_ = kw.pop("gb_format", "f32"), kw.pop("open", False)
    cfg = dataclasses.replace(sg.CONFIGS[room], probe_dims=(8, 4, 8), probe_spacing=4.0,
                              params=dataclasses.replace(sg.CONFIGS[room].params, M=4, **kw))
    scene = sg.make_scene(cfg)
    if open_:
        scene = dataclasses.replace(scene, has_room=False, sky=np.array([1.0, 2.0, 3.0], np.float32))
    out = []
    for lds, grid in ((True, True), (False, True), (False, False)):
        r = gi.Renderer(cfg, seed=5, width=W, height=H, scene=scene, lds=lds, use_grid=grid, gb_format=gbf)
        r.probe.load(*sg.random_probe_textures(r.grid, 3))
        gi.trace_gbuffer(r.dscene, r.camera(0), r.gb[0])
        gi.resample_initial(r.dscene, r.gb[0], r.probe, r.params, r.res[0], r.resid, 5, 1)
        planes = []
        for sp in range(2):
            src, dst = r.res[sp], r.res[sp + 1]
            for t in (dst.y_W, dst.n_wsum, dst.L_M, dst.tag_prim):
                t.fill_(7)                    # every record has to be written
            gi.resample_spatial(r.dscene, r.gb[0], src, r.params, sp, dst, 5, 1)
            planes += [t.view(torch.int32).clone() for t in (dst.y_W, dst.n_wsum, dst.L_M, dst.tag_prim)]
        torch.cuda.synchronize()
        out.append(planes)
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert torch.equal(a, b), f"{int((a != b).sum())} words differ"
