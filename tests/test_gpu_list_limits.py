"""Primitives and pixels at the limits of what the tile forms' primitive lists
can tell apart, against the brute-force loop over all primitives: whatever the
lists leave out must be nothing that a ray can hit, so every bit agrees.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2108_05263_amd import scenegen as sg

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

CFG = dataclasses.replace(sg.CONFIGS["hd"], n_emitters=0, n_spheres=40, n_boxes=37, probe_dims=(4, 2, 4), probe_spacing=8.0)


def _planes(form, scene, W, H, M, lds, edit=None):
    """The pass's output planes as bit patterns: lists (lds) or brute force, no grid in either."""
    from paper_2108_05263_amd import gi
    cfg = dataclasses.replace(CFG, params=dataclasses.replace(CFG.params, M=M))
    r = gi.Renderer(cfg, seed=11, width=W, height=H, scene=scene, lds=lds, use_grid=False)
    r.probe.load(*sg.random_probe_textures(r.grid, 3))
    gi.trace_gbuffer(r.dscene, r.camera(0), r.gb[0])
    if edit is not None:
        edit(r.gb[0])
    res = r.res[0]
    planes = [res.y_W, res.n_wsum, res.L_M, res.tag_prim, r.resid]
    for t in planes:
        t.fill_(7)                            # every record has to be written
    if form == "probe":
        gi.resample_initial(r.dscene, r.gb[0], r.probe, r.params, res, r.resid, 11, 3)
    else:
        mlp = gi.Mlp(cfg.room_lo, cfg.room_hi, precision="bf16", mode="always")
        mlp.init(5)
        ws = gi.initial_mlp_workspace(W, H, M).zero_()
        gi.resample_initial_mlp(r.dscene, r.gb[0], r.probe, mlp, r.params, res, r.resid, ws, 11, 3)
        planes.append(ws)
    torch.cuda.synchronize()
    return [t.view(torch.int32).clone() for t in planes]


def _odd_scene(kind):
    sc = sg.make_scene(CFG)
    prims = sc.prims.copy()
    if kind == "negative":                    # a radius or half extent is squared, or its two ends ordered
        prims[::2, 4:7] *= -1.0
    else:
        types, centre, half = {"slab": ([sg.PRIM_BOX], [16.0, -1.0, 16.0], [np.inf, 0.5, np.inf]),
                               "far": ([sg.PRIM_BOX], [0.0, 0.0, 3e19], [2.9e19, 2.9e19, 2.9e19])}[kind]
        prims = np.concatenate([prims, sg.prim_records(types, [centre], [half], [[0.5] * 3], [[2.0] * 3])])
    return dataclasses.replace(sc, prims=np.ascontiguousarray(prims), has_room=False, sky=np.array([1.0, 2.0, 3.0], np.float32))


@pytest.mark.parametrize("form", ["probe", "cache"])
@pytest.mark.parametrize("kind", ["negative", "slab", "far"])
def test_odd_primitives_stay_in_the_lists(kind, form):
    scene = _odd_scene(kind)
    lists, brute = (_planes(form, scene, 90, 50, 32, lds) for lds in (True, False))
    chosen = brute[3].view(-1, 2)[:, 1]
    odd = (chosen >= 0) & (chosen % 2 == 0) if kind == "negative" else chosen == len(scene.prims) - 1
    assert odd.any(), "the odd primitives are hit"
    for a, b in zip(lists, brute):
        assert torch.equal(a, b), f"{int((a != b).sum())} words differ"


def _odd_pixels(gb):
    gb.nrm_prim[::3, :3] *= -0.5
    gb.nrm_prim[1::7, :3] *= 3.0
    gb.nrm_prim[5::90, :3] *= 1.01            # a tile's only one
    gb.nrm_prim[77, 1] = float("nan")
    gb.pos_depth[123, 0] = float("inf")
    gb.pos_depth[2345, 2] = float("nan")


# normals of other lengths (directions of other lengths, for which the ray
# parameter is no distance) and pixels without a place
@pytest.mark.parametrize("form", ["probe", "cache"])
@pytest.mark.parametrize("open_", [False, True])
def test_odd_pixels_find_the_brute_force_hits(open_, form):
    scene = sg.make_scene(CFG)
    if open_:
        scene = dataclasses.replace(scene, has_room=False, sky=np.array([1.0, 2.0, 3.0], np.float32))
    lists, brute = (_planes(form, scene, 90, 50, 32, lds, _odd_pixels) for lds in (True, False))
    for a, b in zip(lists, brute):
        assert torch.equal(a, b), f"{int((a != b).sum())} words differ"


@pytest.mark.parametrize("form", ["probe", "cache"])
@pytest.mark.parametrize("W,H,M", [(90, 50, 32), (320, 330, 24), (61, 77, 8)])
@pytest.mark.parametrize("values", [(float("nan"), float("inf"), -float("inf")), (3e38, -3e38), (1e19, -1e17)])
def test_scattered_pixels_without_a_place(W, H, M, form, values):
    """One pixel in seven far off, further than FP32 can span, or not a point, along one axis."""
    def edit(gb):
        i = torch.arange(0, gb.pos_depth.shape[0], 7, device="cuda")
        gb.pos_depth[i, 1] = torch.tensor(values, device="cuda")[torch.arange(len(i), device="cuda") % len(values)]

    lists, brute = (_planes(form, sg.make_scene(CFG), W, H, M, lds, edit) for lds in (True, False))
    for a, b in zip(lists, brute):
        assert torch.equal(a, b), f"{int((a != b).sum())} words differ"
