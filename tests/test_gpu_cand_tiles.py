"""The tiled candidate trace of the learned-cache form against the pixel form.

Scenes with GI_OPT_NO_LDS trace one pixel per lane; the tiled form sorts the
rays and tests direction-binned primitive lists, and must leave the same
candidates in the workspace, so every bit of the pass agrees.
"""
import dataclasses

import pytest
import torch

from paper_2108_05263_amd import scenegen as sg

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# tiles of 8x8, 16x8, 16x16 and 32x16 pixels, whole and ragged; one round and
# several, the last one partly filled; both rays-per-thread forms; M on either
# side of the rules; emitter candidates; the gate of AUTO (untrained: probes)
@pytest.mark.parametrize("room,W,H,M,mode,m_light", [
    ("tiny", 64, 64, 8, "always", 0),
    ("tiny", 5, 3, 32, "always", 0),
    ("hd", 65, 33, 7, "always", 0),
    ("hd", 65, 33, 11, "always", 4),
    ("hd", 250, 141, 31, "always", 0),
    ("hd", 1025, 721, 32, "always", 0),
    ("hd", 1283, 721, 13, "always", 0),
    ("hd", 1601, 1283, 9, "always", 0),
    ("hd", 90, 50, 16, "auto", 0),
    ("uhd", 323, 181, 24, "always", 0),
    ("uhd", 1027, 519, 32, "always", 0),
    ("uhd", 90, 50, 23, "always", 0),
    ("uhd", 90, 50, 8, "always", 0),
    ("uhd", 257, 256, 13, "always", 0),        # past the small images' rule: both sides are the pixel form
])
def test_cand_tiles_are_the_pixel_form(room, W, H, M, mode, m_light):
    from paper_2108_05263_amd import gi
    cfg = sg.CONFIGS[room]
    cfg = dataclasses.replace(cfg, probe_dims=(8, 4, 8), probe_spacing=cfg.room_hi[0] / 8,
                              params=dataclasses.replace(cfg.params, M=M, M_light=m_light))
    scene = sg.make_scene(cfg)
    out = []
    for lds in (True, False):
        r = gi.Renderer(cfg, seed=11, width=W, height=H, scene=scene, lds=lds)
        r.probe.load(*sg.random_probe_textures(r.grid, 3))
        gi.trace_gbuffer(r.dscene, r.camera(0), r.gb[0])
        mlp = gi.Mlp(cfg.room_lo, cfg.room_hi, precision="bf16", mode=mode)
        mlp.init(5)
        res, ws = r.res[0], gi.initial_mlp_workspace(W, H, M)
        planes = (res.y_W, res.n_wsum, res.L_M, res.tag_prim, r.resid)
        for t in planes:
            t.fill_(7)
        ws.zero_()
        gi.resample_initial_mlp(r.dscene, r.gb[0], r.probe, mlp, r.params, res, r.resid, ws, 11, 3)
        torch.cuda.synchronize()
        out.append([t.view(torch.int32).clone() for t in planes] + [ws])
    for a, b, name in zip(*out, ("y_W", "n_wsum", "L_M", "tag_prim", "residual", "workspace")):
        assert torch.equal(a, b), f"{name}: {int((a != b).sum())} differ"
