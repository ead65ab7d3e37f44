"""The temporal and shading passes past the small images' rule (65,536 pixels):
every way of reaching the scene at shapes that leave the tiles ragged or few,
with the options that only these forms see there, bit for bit."""
import pytest
import torch

from test_gpu_pass_forms import test_pass_scene_access_is_bit_identical as scene_access

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


# one tile column, less than a wave wide, and a few; one row of tiles
@pytest.mark.parametrize("room,W,H,kw", [
    ("uhd", 5, 13201, {}), ("uhd", 49, 1400, {"gb_format": "f16"}), ("uhd", 433, 157, {"open": True}),
    ("uhd", 4801, 15, {}), ("hd", 9, 7300, {}), ("hd", 333, 201, {"open": True, "gb_format": "f16"}),
])
def test_narrow_and_ragged_images(room, W, H, kw):
    assert W * H > 65536
    scene_access(room, W, H, kw)
