"""The temporal and shading passes' ways of reaching the scene: staged for a
16x16 tile, staged for the 768 threads of a 48x16 tile, and read from global
memory.  Only where the walk reads differs, so every output bit has to agree;
the passes themselves are checked against the oracle by the parity tests.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2108_05263_amd import scenegen as sg

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# edges of both tile widths and of one pixel; both texel and G-buffer formats; an open scene
@pytest.mark.parametrize("room,W,H,kw", [
    ("hd", 17, 33, {}), ("uhd", 1, 1, {}), ("uhd", 48, 16, {}), ("uhd", 49, 17, {"texel": "f16"}),
    ("uhd", 385, 217, {}), ("uhd", 95, 31, {"gb_format": "f16"}), ("uhd", 200, 100, {"open": True}),
    ("glossy", 101, 67, {}),
])
def test_pass_scene_access_is_bit_identical(room, W, H, kw):
    from paper_2108_05263_amd import gi
    kw = dict(kw)
    gbf, open_, texel = kw.pop("gb_format", "f32"), kw.pop("open", False), kw.pop("texel", "f32")
    cfg = sg.CONFIGS[room]
    cfg = dataclasses.replace(cfg, probe_dims=(8, 4, 8), probe_spacing=cfg.room_hi[0] / 8, probe_texel=texel,
                              params=dataclasses.replace(cfg.params, M=4, temporal=True))
    scene = sg.make_scene(cfg)
    if open_:
        scene = dataclasses.replace(scene, has_room=False, sky=np.array([1.0, 2.0, 3.0], np.float32))
    out = []
    for lds in (True, False):
        r = gi.Renderer(cfg, seed=5, width=W, height=H, scene=scene, lds=lds, gb_format=gbf)
        r.probe.load(*sg.random_probe_textures(r.grid, 3))
        cams = [r.camera(0), r.camera(1)]
        for f in (0, 1):
            gi.trace_gbuffer(r.dscene, cams[f], r.gb[f])
            gi.resample_initial(r.dscene, r.gb[f], r.probe, r.params, r.res[f], r.resid, 5, f)
        merged = r.res[2]
        planes = [merged.y_W, merged.n_wsum, merged.L_M, merged.tag_prim]
        for t in planes:
            t.fill_(7)                        # every record has to be written
        gi.resample_temporal(r.dscene, r.gb[1], r.gb[0], cams[0], r.res[1], r.res[0], r.params, merged, 5, 1)
        for src in (r.res[1], merged):
            img = torch.full((W * H, 4), 7.0, device="cuda")
            gi.shade(r.dscene, r.gb[1], r.probe, src, r.resid, r.params, img, seed=5, frame=1)
            planes.append(img)
        if room != "glossy":
            mlp = gi.Mlp(cfg.room_lo, cfg.room_hi, mode="always")
            mlp.init(5)
            img = torch.full((W * H, 4), 7.0, device="cuda")
            gi.shade_mlp(r.dscene, r.gb[1], r.probe, mlp, merged, r.resid, r.params, img, gi.shade_mlp_workspace(W, H))
            planes.append(img)
        torch.cuda.synchronize()
        out.append([t.view(torch.int32).clone() for t in planes])
    for a, b in zip(*out):
        assert torch.equal(a, b), f"{int((a != b).sum())} words differ"
