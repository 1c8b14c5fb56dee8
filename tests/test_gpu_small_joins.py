"""Small images with as many joins as their lines can list: columns staggered
every other row touch two intervals of the line above each; and the sizes where
one launch ends and three begin."""
import numpy as np
import pytest

import oracle
from paper_1708_08180_amd import workloads as wl
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

# the last three rows: the first and last sizes of one launch and of three
SHAPES = [(120, 160), (128, 192), (192, 128), (129, 130), (128, 256), (512, 64), (127, 250),
          (320, 64), (321, 64), (2, 8192), (2, 8193), (32, 512), (32, 513),
          (32, 640), (32, 641), (2, 10240), (2, 10241), (46, 384), (46, 449),
          (48, 576), (48, 577), (448, 64), (449, 64)]


def _staggered(H, W, step=2):
    yy, xx = np.indices((H, W))
    return ((xx + yy // step) % 2).astype(np.uint8)


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("shape", SHAPES)
def test_many_joins(shape, conn):
    import torch
    from paper_1708_08180_amd import binding

    images = [_staggered(*shape, step) for step in (1, 2, 3)] + [wl.bernoulli(*shape, p, 4400) for p in (0.4, 0.6)]
    for k, img in enumerate(images):
        out = binding.label(to_dev(img), conn)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy().view(np.uint32), oracle.label(img, conn)), k


@pytest.mark.parametrize("shape", [(120, 160), (128, 192)])
def test_joins_that_fit_the_list(shape):
    # 3 to 4 times the three phases' time when the list was too short for them
    import torch
    from paper_1708_08180_amd import binding

    d = to_dev(_staggered(*shape))
    out = torch.empty(shape, dtype=torch.int32, device="cuda")

    def us(config):
        best = 1e9
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(50):
                binding.label(d, 8, out=out, config=config)
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) * 20.0)
        return best

    one, three = us(None), us((32, 8))
    say("%dx%d one launch %.1f us, three %.1f" % (shape + (one, three)))
    assert one < 2.0 * three
