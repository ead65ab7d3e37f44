"""The spatial pass's 8x8 tiles for images of few pixels against the wider
tiles of larger ones: the first rows of an image, taken as a smaller image of
the same width, keep every bit up to a search radius from its last row."""
import dataclasses

import pytest
import torch

from paper_2108_05263_amd import scenegen as sg
from test_gpu_spatial_forms import test_spatial_scene_access_is_bit_identical as scene_access

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.fixture(scope="module")
def gi():
    from paper_2108_05263_amd import gi as g
    g.load()
    return g


# every scene form (staged, staged wide, too large to stage beside it), the
# glossy target, no and the most neighbours; the largest image of the rule
@pytest.mark.parametrize("room,k,W,H", [("tiny", 5, 256, 256), ("hd", 8, 250, 141), ("hd", 0, 100, 65), ("uhd", 5, 255, 257),
                                        ("glossy", 5, 203, 151)])
def test_small_image_tiles_are_bit_identical(gi, room, k, W, H):
    cfg = dataclasses.replace(sg.CONFIGS[room], probe_dims=(4, 4, 4), probe_spacing=sg.CONFIGS[room].room_hi[0] / 4,
                              params=dataclasses.replace(sg.CONFIGS[room].params, M=4, k=k))
    tall, scene = 65536 // W + 40, sg.make_scene(cfg)
    assert W * H <= 65536 < W * tall
    big, small = (gi.Renderer(cfg, seed=5, width=W, height=h, scene=scene) for h in (tall, H))
    big.probe.load(*sg.random_probe_textures(big.grid, 3))
    gi.trace_gbuffer(big.dscene, big.camera(0), big.gb[0])
    gi.trace_gbuffer(small.dscene, small.camera(0), small.gb[0])
    gi.resample_initial(big.dscene, big.gb[0], big.probe, big.params, big.res[0], big.resid, 5, 1)
    for a, b in ((small.gb[0], big.gb[0]), (small.res[0], big.res[0])):
        for name, t in vars(a).items():
            if torch.is_tensor(t):
                t.copy_(getattr(b, name)[:W * H])
    rows = (H - int(cfg.params.radius) - 2) * W
    out = []
    for r in (big, small):
        dst = r.res[1]
        planes = (dst.y_W, dst.n_wsum, dst.L_M, dst.tag_prim)
        for t in planes:
            t.fill_(7)                        # every record has to be written
        gi.resample_spatial(r.dscene, r.gb[0], r.res[0], r.params, 0, dst, 5, 1)
        out.append([t.view(torch.int32)[:rows].clone() for t in planes])
    for a, b in zip(*out):
        assert torch.equal(a, b), f"{int((a != b).sum())} words differ"


# the larger images' forms, past the smaller ones' rule
@pytest.mark.parametrize("room,W,H,kw", [("hd", 333, 201, {}), ("glossy", 257, 257, {"k": 8}), ("uhd", 337, 197, {"k": 8})])
def test_larger_images_scene_access(gi, room, W, H, kw):
    scene_access(gi, room, W, H, kw)
