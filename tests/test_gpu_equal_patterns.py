"""Equal-value labeling of patterns that hook every run: as many joins as a tile
can list (checkerboards and staggered columns, whose runs touch two runs of the
row above), and chains as deep as a tile (columns)."""
import numpy as np
import pytest

import oracle
from tests.gpu_util import say, to_dev

pytestmark = pytest.mark.gpu

PATTERNS = {
    "checkerboard": lambda y, x: (x + y) % 2,
    "three values": lambda y, x: (x + y) % 3,
    "staggered": lambda y, x: (x + y // 2) % 2,
    "columns": lambda y, x: x % 2,
    "columns joined below": lambda y, x: (x % 2 == 0) | (y % 64 == 63),
    "diagonal pairs": lambda y, x: (x // 2 + y) % 2,
}


def _image(name, H, W):
    yy, xx = np.indices((H, W))
    return PATTERNS[name](yy, xx).astype(np.uint8)


@pytest.mark.parametrize("conn", [4, 8])
@pytest.mark.parametrize("name", sorted(PATTERNS))
def test_patterns(name, conn):
    import torch
    from paper_1708_08180_amd import binding

    for H, W in ((64, 64), (67, 131), (300, 257)):
        img = _image(name, H, W)
        want = oracle.label_equal(img, conn)
        for config in (None, (16, 4), (32, 2), (32, 8), (64, 4), (64, 8)):
            out = binding.label_equal(to_dev(img), conn, config=config)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy().view(np.uint32), want), (H, W, config)


def _us(img, conn):
    import torch
    from paper_1708_08180_amd import binding

    out = torch.empty(tuple(img.shape), dtype=torch.int32, device="cuda")
    best = 1e9
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            binding.label_equal(img, conn, out=out)
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 100.0)
    return best


def _against_noise(name, conn):
    H, W = 4096, 4096
    noise = to_dev(np.random.default_rng(5).integers(0, 2, (H, W), dtype=np.uint8))
    t, ref = _us(to_dev(_image(name, H, W)), conn), _us(noise, conn)
    say("%s %.1f us, noise of two values %.1f" % (name, t, ref))
    return t / ref


def test_joins_that_fit_the_list():
    # 3.6 times the time of noise when the list was too short for them
    assert _against_noise("checkerboard", 8) < 2.0


def test_deep_chains():
    # 1.6 times the time of noise when every run walked up the whole tile
    assert _against_noise("columns", 4) < 1.4
