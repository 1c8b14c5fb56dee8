"""Image rows at any byte address and of any length: the 16-byte row loads
against the oracle (bit for bit), where a row's end cuts a chunk, where rows
are shorter than one chunk, and where neither the image nor its pitch is
aligned."""
import numpy as np
import pytest

import oracle
from paper_1708_08180_amd import workloads as wl
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

WIDTHS = (1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 79, 80, 81, 127, 129, 191)


def _view(img, offset, pad):
    """`img` on the device as a view `offset` bytes into rows `pad` bytes longer."""
    import torch

    H, W = img.shape
    big = torch.full((H, offset + W + pad), 9, dtype=torch.uint8, device="cuda")
    big[:, offset:offset + W] = torch.from_numpy(img).cuda()
    return big[:, offset:offset + W]


@pytest.mark.parametrize("offset,pad", [(0, 0), (0, 1), (1, 0), (3, 2), (7, 9), (15, 17)])
def test_row_loads(offset, pad):
    import torch
    from paper_1708_08180_amd import binding

    for k, W in enumerate(WIDTHS):
        img = wl.bernoulli(37, W, 0.55, 7100 + k, fg=200)
        d = _view(img, offset, pad)
        say("row loads W=%d offset=%d pad=%d" % (W, offset, pad))
        for conn in (4, 8):
            got = binding.label(d, conn)
            eq = binding.label_equal(d, conn)
            torch.cuda.synchronize()
            assert np.array_equal(got.cpu().numpy().view(np.uint32), oracle.label(img, conn))
            assert np.array_equal(eq.cpu().numpy().view(np.uint32), oracle.label_equal(img, conn))
        v = d.unsqueeze(0)
        got = binding.label3d(v, 26)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy().view(np.uint32), oracle.label3d(img[None], 26))
