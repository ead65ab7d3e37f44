"""The tiled candidate trace past the size at which its rule counts the
primitives, on either side of the rule, against the pixel form."""
import pytest
import torch

from test_gpu_cand_tiles import test_cand_tiles_are_the_pixel_form as cand_forms

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("M", [29, 30])
def test_large_image_of_many_primitives(M):
    cand_forms("uhd", 1501, 1003, M, "always", 0)
