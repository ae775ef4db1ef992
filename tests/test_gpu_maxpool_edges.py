"""Max pooling in 16-byte granules against PyTorch on the CPU, bit for bit (a maximum rounds nothing): channel
counts that are and are not whole granules, windows of three and others, rows that end inside a block."""
import pytest

from paper_2507_17301_amd import binding as nm
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("b,h,w,c,k,stride,pad", [
    (1, 3, 3, 8, 3, 2, 1), (2, 13, 9, 64, 3, 2, 1), (3, 7, 33, 72, 3, 1, 1), (1, 5, 5, 4, 3, 2, 1), (2, 9, 9, 6, 3, 2, 1),
    (1, 8, 8, 16, 2, 2, 0), (2, 11, 12, 24, 5, 3, 2), (1, 6, 300, 8, 1, 1, 0), (1, 1, 1, 2048, 3, 2, 1)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_maxpool_edges(b, h, w, c, k, stride, pad, dtype):
    import torch
    say(f"maxpool {b} {h} {w} {c} {k} {stride} {pad} {dtype}")
    g = torch.Generator().manual_seed(7)
    x = torch.randn((b, h, w, c), generator=g).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    x[0, 0, 0, 0] = float("-inf")
    y = nm.nm_maxpool2d(x.cuda(), k, stride, pad)
    torch.cuda.synchronize()
    ref = torch.nn.functional.max_pool2d(x.float().permute(0, 3, 1, 2), k, stride, pad).permute(0, 2, 3, 1)
    assert torch.equal(y.float().cpu(), ref)
