"""One row of pixels so long that a launch does not hold the threads that the
link runs with elsewhere."""
import pytest

from tests.gpu_util import say

pytestmark = pytest.mark.gpu


def test_long_row_narrow_link():
    import torch
    from paper_1708_08180_amd import binding

    W = 64 * (2 ** 32 // 256) + 1001  # one tile more than 4 wavefronts each can take, and a ragged one
    need = binding.workspace_size(1, W, (32, 1))
    if torch.cuda.mem_get_info()[0] < need + 8 * W + (4 << 30):
        pytest.skip("needs %d GB of device memory" % ((need + 8 * W) >> 30))
    say("1 x %d, workspace %d GB" % (W, need >> 30))
    g = torch.Generator(device="cuda").manual_seed(77)
    img = torch.empty((1, W), dtype=torch.uint8, device="cuda").random_(0, 2, generator=g)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    out = binding.label(img, 8, config=(32, 1), workspace=ws)
    torch.cuda.synchronize()
    # a run's pixels hold 1 + its first column
    part, before, start = 1 << 26, 0, 0
    for x0 in range(0, W, part):
        m = img[0, x0:x0 + part].to(torch.bool)
        left = torch.cat([torch.tensor([bool(before)], device="cuda"), m[:-1]])
        at = torch.arange(x0 + 1, x0 + 1 + m.numel(), device="cuda") * (m & ~left)
        at[0] = torch.maximum(at[0], torch.tensor(start, device="cuda"))
        first = at.cummax(0).values
        assert torch.equal(out[0, x0:x0 + part].to(torch.int64), torch.where(m, first, torch.zeros_like(first))), x0
        before, start = int(m[-1]), int(first[-1])
