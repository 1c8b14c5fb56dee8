"""Statistics of label images in the blocks of 32 and 64 rows that small images
take, and at the sizes where they end."""
import numpy as np
import pytest

import oracle
from paper_1708_08180_amd import workloads as wl
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

# blocks of 32 rows: the smallest, one row and column past a block, the most
# (96; 128 of two rows); of 64 rows: the fewest, ragged, the most (128)
SHAPES = [(1, 129), (32, 128), (33, 129), (96, 4096), (64, 8192), (3072, 128),
          (97, 4096), (65, 8192), (65, 8193), (513, 1800), (3073, 128), (1024, 1024), (1025, 1024)]


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("shape", SHAPES)
def test_small_blocks(shape, conn):
    import torch
    from paper_1708_08180_amd import binding

    H, W = shape
    yy, xx = np.indices(shape)
    images = [wl.bernoulli(H, W, p, 9100) for p in (0.3, 0.6)]
    images += [((xx % 2) * (yy % 2)).astype(np.uint8), ((yy // 24 + xx // 40) % 2).astype(np.uint8), np.ones(shape, np.uint8)]
    for k, img in enumerate(images):
        got = binding.component_stats(binding.label(to_dev(img), conn))
        want = oracle.stats(img, conn)
        assert len(got) == len(want), k
        for f in ("label", "area", "x_min", "y_min", "x_max", "y_max", "sum_x", "sum_y"):
            assert np.array_equal(np.asarray(got[f]).astype(np.uint64), np.asarray(want[f]).astype(np.uint64)), (k, f)
    torch.cuda.synchronize()


def test_dense_small_image_is_spread():
    # 4.5 times the time of an empty image when one workgroup added it all up
    import torch
    from paper_1708_08180_amd import binding

    lib = binding.load_library()
    s = torch.cuda.current_stream().cuda_stream
    rec = torch.zeros((1 << 14, 10), dtype=torch.int32, device="cuda")
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")

    def us(img):
        lab = binding.label(to_dev(img), 4)
        best = 1e9
        for _ in range(10):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(50):
                assert lib.ccl_component_stats(lab.data_ptr(), 128, 128, rec.data_ptr(), 1 << 14, cnt.data_ptr(), s) == 0
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 20.0)
        return best

    dense, empty = us(wl.bernoulli(128, 128, 0.5, 9101)), us(np.zeros((128, 128), np.uint8))
    say("128x128: noise %.1f us, empty %.1f" % (dense, empty))
    assert dense < 3.0 * empty
