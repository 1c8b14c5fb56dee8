"""Statistics of a label image at the sizes where the accumulation's blocks
(128 x 128 pixels, strips of 16 rows), the root words and the record numbering
begin and end, field by field against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1708_08180_amd import workloads as wl
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def _check(img, conn, what):
    import torch
    from paper_1708_08180_amd import binding

    say("stats %s %s conn=%d" % (what, img.shape, conn))
    lab = binding.label(torch.from_numpy(img).cuda(), conn)
    got = binding.component_stats(lab)
    want = oracle.stats(img, conn)
    assert len(got) == len(want)
    for f in ("label", "area", "x_min", "y_min", "x_max", "y_max", "sum_x", "sum_y"):
        assert np.array_equal(np.asarray(got[f]).astype(np.uint64), np.asarray(want[f]).astype(np.uint64)), f


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("shape", [(1, 1), (15, 127), (16, 128), (17, 129), (127, 64), (128, 65), (257, 191), (31, 513),
                                   (600, 300)])
def test_block_edges(shape, conn):
    H, W = shape
    for k, p in enumerate((0.2, 0.5, 0.7)):
        _check(wl.bernoulli(H, W, p, 8700 + k), conn, "noise %.1f" % p)
    yy, xx = np.indices((H, W))
    _check(((yy // 24 + xx // 40) % 2).astype(np.uint8), conn, "blocks")
    _check(np.ones((H, W), np.uint8), conn, "full")


def test_many_blocks():
    # more blocks of root words than the self-summing record numbering takes,
    # and more components per block than its table holds
    img = np.zeros((8192, 4352), np.uint8)
    img[::2, ::2] = 1
    img[-2, :] = 1
    img[:, 4000] = 1
    _check(img, 4, "lattice")
    # one row of words per image row: 2048 * 256 words and a few more
    img = np.zeros((262144 + 300, 65), np.uint8)
    img[5::97, 3:60] = 1
    img[200::301, :] = 1
    _check(img, 8, "tall")


@pytest.mark.parametrize("conn", [4, 8])
def test_blocks_share_a_table(conn):
    # workgroups of several blocks: one flush at the end (large components), a
    # flush in between (many components), both in one column of blocks
    H, W = 4097 + 128, 4096 + 70
    img = np.zeros((H, W), np.uint8)
    img[: H // 2] = wl.bernoulli(H // 2, W, 0.62, 8800)
    img[H // 2:, ::2] = 1
    img[H // 2 + 1::9] = 0
    _check(img, conn, "several blocks")
