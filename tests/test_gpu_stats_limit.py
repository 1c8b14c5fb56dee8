"""Component statistics of label images at the documented size limit
(H * W <= 2^32 - 1), where 32-bit pixel indices of the columns right of the
image wrap around and the last pixel's label is 2^32 - 1."""
import numpy as np
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu

# H * W = 2^32 - 1, and two ragged widths within one row word of 2^32
SHAPES = [(65535, 65537), (66076419, 65), (33818640, 127)]


def _zeros(shape):
    import torch

    need = 4 * shape[0] * shape[1] + (4 << 30)
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip("needs %d GB of device memory" % (need >> 30))
    return torch.zeros(shape, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("shape", SHAPES)
def test_background_has_no_components(shape):
    from paper_1708_08180_amd import binding

    say("limit %s background" % (shape,))
    assert len(binding.component_stats(_zeros(shape))) == 0
    binding.shutdown()


@pytest.mark.parametrize("shape", SHAPES)
def test_last_pixel_is_a_component(shape):
    # its label is H * W, 2^32 - 1 for the first shape
    from paper_1708_08180_amd import binding

    H, W = shape
    lab = _zeros(shape)
    lab.view(-1)[-1] = np.uint32(H * W).view(np.int32).item()
    lab[H // 2, 1:9] = np.uint32(H // 2 * W + 2).view(np.int32).item()
    say("limit %s last pixel" % (shape,))
    got = binding.component_stats(lab)
    y = H // 2
    want = [(y * W + 2, 8, 1, y, 8, y, 36, 8 * y), (H * W, 1, W - 1, H - 1, W - 1, H - 1, W - 1, H - 1)]
    assert [tuple(int(v) for v in r) for r in got] == want
    binding.shutdown()
