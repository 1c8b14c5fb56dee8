"""The tile-local merge over two-row bands where its rules can go wrong, bit
for bit against the oracle: a component whose root interval has no top-row
pixel while other intervals of its band do (its smallest pixel is theirs), the
most intervals per band, the most joins per tile, and bands cut by the image's
last row."""
import numpy as np
import pytest

import oracle
from paper_1708_08180_amd import workloads as wl
from tests.gpu_util import gpu_label, say

pytestmark = pytest.mark.gpu

CONFIGS = [None, (16, 1), (16, 8), (32, 4), (64, 1), (64, 2), (64, 16), (128, 2), (128, 8)]


def _check(img, conn, config, what):
    say("local merge %s %s conn=%d config=%s" % (what, img.shape, conn, config))
    got = gpu_label(img, conn, config=config)
    assert np.array_equal(got, oracle.label(img, conn)), what


def combs(H, W):
    """Per band: a bottom-row pixel at the left, top-row pixels at its right,
    all joined by a full row three rows below."""
    img = np.zeros((H, W), np.uint8)
    for y in range(0, H - 6, 6):
        img[y + 1:y + 4, 3::23] = 1
        img[y:y + 4, 9::23] = 1
        img[y:y + 4, 15::23] = 1
        img[y + 3, :] = 1
    return img


def alternating(H, W, p_even, p_odd, seed):
    rng = wl.rng_for(seed)
    img = rng.random((H, W))
    p = np.where(np.arange(H) % 2 == 0, p_even, p_odd)[:, None]
    return (img < p).astype(np.uint8)


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("config", CONFIGS)
def test_band_roots(conn, config):
    for H, W in ((131, 200), (64, 64), (129, 65)):
        _check(combs(H, W), conn, config, "combs")
        for k, (pe, po) in enumerate(((0.1, 0.6), (0.6, 0.1), (0.25, 0.75), (0.5, 0.5))):
            _check(alternating(H, W, pe, po, 8100 + k), conn, config, "alternating %.2f %.2f" % (pe, po))


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("config", CONFIGS)
def test_most_intervals(conn, config):
    H, W = 129, 130
    yy, xx = np.indices((H, W))
    for what, img in (("checkerboard", (xx + yy) % 2 == 0), ("columns", xx % 2 == 0),
                      ("staggered", (xx + (yy // 2)) % 2 == 0), ("diagonals", (xx + yy) % 3 == 0),
                      ("zigzag", ((xx + yy) % 4 < 2) & (yy % 4 != 3))):
        img = img.astype(np.uint8)
        _check(img, conn, config, what)
        img[H - 1, :] = 1  # joined at the very end
        _check(img, conn, config, what + ", joined")
