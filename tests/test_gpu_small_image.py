"""Images labeled in one launch (up to 256 lines of two rows and 64 columns)
and the first ones that are not, bit for bit against the oracle; the calls that
keep the three phases (a configuration from the caller or the tuning table)
give the same labels, with the same checks of a caller's workspace."""
import numpy as np
import pytest

import oracle
from paper_1708_08180_amd import workloads as wl
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

# lines: 1, 1, 2, .., the most (256) as a square, a row, a column, and one more
SHAPES = [(1, 1), (2, 64), (1, 65), (3, 64), (5, 127), (63, 129), (64, 192), (120, 160), (128, 256), (127, 250),
          (2, 16384), (1, 16300), (512, 64), (511, 1), (170, 192), (130, 256), (2, 16385), (513, 64)]


def _label(img, conn, fn, **kw):
    import torch

    out = fn(to_dev(img, kw.pop("pad", 0)), conn, **kw)
    torch.cuda.synchronize()
    return out.cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_images(shape, conn):
    from paper_1708_08180_amd import binding

    H, W = shape
    yy, xx = np.indices((H, W))
    images = [wl.bernoulli(H, W, p, 6600 + k) for k, p in enumerate((0.15, 0.5, 0.62, 0.85))]
    images += [((xx + yy) % 2).astype(np.uint8), (xx % 2).astype(np.uint8), np.ones((H, W), np.uint8),
               np.zeros((H, W), np.uint8), wl.serpentine(H, W), ((yy % 4 == 1) | (xx % 7 == 3)).astype(np.uint8)]
    for k, img in enumerate(images):
        say("small %dx%d conn=%d image %d" % (H, W, conn, k))
        want = oracle.label(img, conn)
        assert np.array_equal(_label(img, conn, binding.label), want)
        assert np.array_equal(_label(img, conn, binding.label_plain, pad=5), want)
        assert np.array_equal(_label(img, conn, binding.label_noalloc), want)
        assert np.array_equal(_label(img, conn, binding.label, config=(32, 4)), want)


def test_small_image_words():
    """Touches across the 64-column words: straight, diagonal, and through the
    other row of a band only."""
    from paper_1708_08180_amd import binding

    for conn in (4, 8):
        for a in range(16):
            for b in range(16):
                img = np.zeros((8, 130), np.uint8)
                for i in range(4):
                    img[2 + i, 63] = (a >> i) & 1
                    img[2 + i, 64] = (b >> i) & 1
                assert np.array_equal(_label(img, conn, binding.label), oracle.label(img, conn)), (conn, a, b)


def test_small_image_workspace_checks():
    import torch
    from paper_1708_08180_amd import binding

    img = to_dev(wl.bernoulli(64, 64, 0.5, 1))
    need = binding.workspace_size(64, 64)
    with pytest.raises(binding.CclError):
        binding.label(img, 8, workspace=torch.empty(need - 1, dtype=torch.uint8, device="cuda"))
    out = binding.label(img, 8, workspace=torch.empty(need, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), oracle.label(img.cpu().numpy(), 8))


def test_small_image_tuned():
    from paper_1708_08180_amd import binding

    img = wl.bernoulli(120, 160, 0.5, 2)
    try:
        binding.autotune(to_dev(img), 8, reps=1)
        assert np.array_equal(_label(img, 8, binding.label), oracle.label(img, 8))
    finally:
        binding.tuning_clear()
