"""The kernels and grids that calls launch, over the sizes the entry points
accept: HIP refuses a launch of 2^32 threads or more, so images of very few
rows or columns, which have many tiles for their pixels, decide what still
fits.  Runs without a GPU (launches are recorded, not made)."""
import pytest

from tests.launches import COUNT, IMG, LABELS, OUT, record


def _plain(H, W, conn=8, cfg=None):
    return ("ccl_label_2d_ex", [IMG, H, W, W, conn, LABELS, None, 0, cfg, None])


def _equal(H, W, conn=8, cfg=None):
    return ("ccl_label_2d_equal", [IMG, H, W, W, conn, LABELS, cfg, None])


def _accepted(results):
    for rc, launches in results:
        assert rc == 0 and launches and not any(l[4] for l in launches), (rc, launches)


def test_equal_value_thin_images(tmp_path):
    # the most tiles of 64 rows that four wavefronts each can take
    most = (2 ** 32 - 1) // 256
    res = record([_equal(1, 64 * most), _equal(64 * most, 1, 4), _equal(1, 64 * (most // 2)), _equal(2160, 3840)], tmp_path)
    _accepted(res)
    assert [ls[0][3] for _, ls in res] == [256, 256, 512, 512]
