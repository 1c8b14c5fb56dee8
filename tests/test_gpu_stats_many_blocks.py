"""Statistics of a label image of so many blocks that a workgroup takes eight of
them below each other, the most: components that span all eight, and so many
small ones that its table is flushed in between."""
import numpy as np

import pytest

import oracle
from paper_1708_08180_amd import workloads as wl
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("conn", [4, 8])
def test_eight_blocks_per_workgroup(conn):
    from paper_1708_08180_amd import binding

    H = W = 8192 + 64  # 65 x 65 blocks of 128 x 128, the last row and column half filled
    img = np.zeros((H, W), np.uint8)
    img[:, : W // 3] = 1                                            # one component over all blocks
    img[:, W // 3 + 2: W // 2] = wl.bernoulli(H, W // 2 - W // 3 - 2, 0.62, 9200)
    img[::2, W // 2 + 1:: 2] = 1                                    # isolated pixels
    img[1024 + 512: 2048 + 512, W // 2 + 2:] = 1                    # large, across two workgroups
    img[3000:, W // 2 + 2: W // 2 + 2 + 64 * 20] = wl.smoothed_noise(H - 3000, 64 * 20, 9.0, 9201)
    say("eight blocks conn=%d" % conn)
    got = binding.component_stats(binding.label(to_dev(img), conn))
    want = oracle.stats(img, conn)
    assert len(got) == len(want)
    for f in ("label", "area", "x_min", "y_min", "x_max", "y_max", "sum_x", "sum_y"):
        assert np.array_equal(np.asarray(got[f]).astype(np.uint64), np.asarray(want[f]).astype(np.uint64)), f
