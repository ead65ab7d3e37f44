"""The temporal pass of images of few pixels against the FP64 oracle, on the
oracle's own inputs, at the edges of its 8x8 tiles and at its largest image
(the staged and the global scene are compared bit for bit elsewhere)."""
import dataclasses

import pytest
import torch

import oracle as o
from paper_2108_05263_amd import scenegen as sg

from helpers import compare_reservoirs

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("W,H,unbiased,lds", [(9, 7, 1, True), (64, 40, 1, False), (65, 33, 0, True), (256, 256, 1, True)])
def test_small_temporal_pass(W, H, unbiased, lds):
    from paper_2108_05263_amd import gi
    cfg = sg.CONFIGS["tiny"]
    cfg = dataclasses.replace(cfg, params=dataclasses.replace(cfg.params, M=4, k=2, n_spatial=1, temporal=True,
                                                              unbiased=unbiased))
    sc, grid = sg.make_scene(cfg), sg.make_probe_grid(cfg)
    irr, dep = sg.random_probe_textures(grid, 3)
    seq, cams = o.Sequence(sc, grid, irr, dep, cfg.params, 1), [sg.make_camera(cfg, f, W, H) for f in (0, 1)]
    st = [seq.frame(c, f)[1] for f, c in enumerate(cams)]
    ds = gi.DeviceScene(sc, cfg.grid_res, lds=lds)
    gb, gbp = gi.GBuffer(W, H), gi.GBuffer(W, H)
    cur, hist, out = (gi.Reservoirs(W, H) for _ in range(3))
    gb.load_records(st[1]["gbuffer"])
    gbp.load_records(st[0]["gbuffer"])
    cur.load_records(st[1]["initial"])
    hist.load_records(st[0]["spatial0"])
    for t in (out.y_W, out.n_wsum, out.L_M, out.tag_prim):
        t.fill_(7)                            # every record has to be written
    gi.resample_temporal(ds, gb, gbp, cams[0], cur, hist, cfg.params, out, 1, 1)
    g = st[1]["gbuffer"]
    active = (g[:, 13] != o.MISS) & (g[:, 6:9].max(1) > 0)
    compare_reservoirs(out.to_records(), st[1]["temporal"], active, label=f"temporal {W}x{H}")
