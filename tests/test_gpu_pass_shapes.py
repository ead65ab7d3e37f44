"""The temporal and shading passes past the small images' rule (65,536 pixels):
every way of reaching the scene at shapes that leave the tiles ragged or few,
and the temporal pass's options there, against the oracle and against the
small images' form."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle as o
from paper_2108_05263_amd import scenegen as sg
from helpers import compare_reservoirs
from test_gpu_pass_forms import test_pass_scene_access_is_bit_identical as scene_access

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

SKY = np.array([1.0, 2.0, 3.0], np.float32)


# one tile column, less than a wave wide, and a few; one row of tiles
@pytest.mark.parametrize("room,W,H,kw", [
    ("uhd", 5, 13201, {}), ("uhd", 49, 1400, {"gb_format": "f16"}), ("uhd", 433, 157, {"open": True}),
    ("uhd", 4801, 15, {}), ("hd", 9, 7300, {}), ("hd", 333, 201, {"open": True, "gb_format": "f16"}),
])
def test_narrow_and_ragged_images(room, W, H, kw):
    assert W * H > 65536
    scene_access(room, W, H, kw)


# the 16x16 and the 48x16 tiles, and the scene from global memory, on the oracle's own inputs
@pytest.mark.parametrize("room,W,H,lds", [("hd", 333, 201, True), ("uhd", 337, 197, True), ("hd", 333, 201, False)])
@pytest.mark.parametrize("open_,kw", [(False, {"unbiased": 0}), (True, {}), (True, {"unbiased": 0}),
                                      (False, {"subsample": 2, "m_cap": 1.3})])
def test_large_temporal_pass(room, W, H, lds, open_, kw):
    from paper_2108_05263_amd import gi
    cfg = sg.CONFIGS[room]
    cfg = dataclasses.replace(cfg, probe_dims=(4, 2, 4), probe_spacing=cfg.room_hi[0] / 4,
                              params=dataclasses.replace(cfg.params, M=2, k=1, n_spatial=1, temporal=True, **kw))
    sc, grid = sg.make_scene(cfg), sg.make_probe_grid(cfg)
    if open_:
        sc = dataclasses.replace(sc, has_room=False, sky=SKY)
    seq, cams = o.Sequence(sc, grid, *sg.random_probe_textures(grid, 3), cfg.params, 1), [sg.make_camera(cfg, f, W, H) for f in (0, 1)]
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
    compare_reservoirs(out.to_records(), st[1]["temporal"], active, label=f"temporal {room} {W}x{H}")


# The first rows of an image, taken as a smaller image.  Its camera is the
# large one's sheared, so that a row's centre projects to the same row; with
# the frame's own vertices as the previous ones every pixel then meets its own
# history in both, and every bit has to agree.
@pytest.mark.parametrize("room,W,H,open_,unbiased,gb_format", [
    ("tiny", 256, 256, False, 1, "f32"), ("hd", 250, 141, False, 1, "f32"), ("hd", 101, 77, True, 0, "f16"),
    ("uhd", 255, 257, False, 1, "f32"), ("uhd", 250, 141, True, 1, "f16"), ("uhd", 99, 101, False, 0, "f32"),
])
def test_small_temporal_tiles_are_the_large_ones(room, W, H, open_, unbiased, gb_format, odd=False):
    from paper_2108_05263_amd import gi
    cfg = sg.CONFIGS[room]
    cfg = dataclasses.replace(cfg, probe_dims=(4, 4, 4), probe_spacing=cfg.room_hi[0] / 4,
                              params=dataclasses.replace(cfg.params, M=4, temporal=True, unbiased=unbiased))
    tall, scene = 65536 // W + 40, sg.make_scene(cfg)
    assert W * H <= 65536 < W * tall
    if open_:
        scene = dataclasses.replace(scene, has_room=False, sky=SKY)
    big, small = (gi.Renderer(cfg, seed=5, width=W, height=h, scene=scene, gb_format=gb_format) for h in (tall, H))
    big.probe.load(*sg.random_probe_textures(big.grid, 3))
    cam = big.camera(0)
    share, T = H / tall, cam.tan_half_fovy
    crop = dataclasses.replace(cam, up=(cam.up - T * (1.0 - share) * cam.fwd).astype(np.float32), tan_half_fovy=T * share, height=H)
    for f in (0, 1):
        gi.trace_gbuffer(big.dscene, cam, big.gb[f])
        gi.resample_initial(big.dscene, big.gb[f], big.probe, big.params, big.res[f], big.resid, 5, f)
    big.gb[0].pos_depth[::5, 3] *= 1.5        # a previous vertex that the depth test refuses
    if odd:
        big.gb[0].albedo[::7, 1] = float("nan")
        big.gb[0].pos_depth[3::11, 1] = float("inf")
    for f in (0, 1):
        for a, b in ((small.gb[f], big.gb[f]), (small.res[f], big.res[f])):
            for name, t in vars(a).items():
                if torch.is_tensor(t):
                    t.copy_(getattr(b, name)[:W * H])
    out = []
    for r, c in ((big, cam), (small, crop)):
        dst = r.res[2]
        planes = (dst.y_W, dst.n_wsum, dst.L_M, dst.tag_prim)
        for t in planes:
            t.fill_(7)                        # every record has to be written
        gi.resample_temporal(r.dscene, r.gb[1], r.gb[0], c, r.res[1], r.res[0], r.params, dst, 5, 1)
        out.append([t.view(torch.int32)[:W * H].clone() for t in planes])
    merged = (out[0][2][:, 3] == 8).sum() / (out[0][2][:, 3] > 0).sum()
    assert 0.7 < merged < 0.9, "four of five pixels take over their history"
    for a, b in zip(*out):
        assert torch.equal(a, b), f"{int((a != b).sum())} words differ"


# previous vertices that are no numbers: a target that is none counts as support in every form
@pytest.mark.parametrize("room,W,H", [("hd", 250, 141), ("uhd", 99, 101)])
def test_previous_vertices_of_no_number(room, W, H):
    test_small_temporal_tiles_are_the_large_ones(room, W, H, False, 1, "f32", odd=True)
