"""The 1x1 bf16 kernel that walks the output channels over resident pixels: the sums of the strip-per-tap form, in its order, so the
same bits, at the edges of tiles, of groups of 256 channels and of the walk."""
import numpy as np
import pytest

from paper_2507_17301_amd import binding as nm
from gpu_util import say

pytestmark = pytest.mark.gpu

# batch, H, W, Cin, Cout, stride, N, M, T, residual, bias: one pixel; one to four chunks; parts of a row block, of a group of 256
# channels and of a tile; walks of one to nine groups, whole and shared by several workgroups
CASES = [(1, 1, 1, 64, 16, 1, 2, 4, 16, False, True), (1, 7, 9, 128, 264, 1, 1, 4, 16, True, True), (3, 13, 11, 192, 520, 2, 2, 8, 32, True, False),
         (2, 8, 8, 256, 1024, 1, 2, 4, 16, True, True), (70, 14, 13, 64, 2056, 1, 2, 4, 16, False, True), (130, 14, 14, 256, 776, 1, 2, 8, 48, True, True),
         (9, 28, 27, 128, 512, 2, 1, 8, 16, True, True),
         # two and three chunks whose workgroups walk: all four groups and, in tiles of 64 pixels, all three; two of four at a time
         (130, 14, 14, 128, 776, 1, 2, 4, 16, True, True), (130, 14, 14, 192, 520, 1, 2, 8, 16, True, True),
         (64, 14, 13, 192, 1016, 1, 1, 4, 16, True, False), (66, 14, 13, 128, 1000, 1, 2, 4, 16, False, True)]


def walk(pixels, cout, blocks):
    """Groups of 256 output channels that a workgroup of 16 `blocks` pixels walks."""
    tiles, groups = -(-pixels // (16 * blocks)), -(-cout // 256)
    parts = -(-384 // tiles)
    return 1 if parts >= groups else -(-groups // parts)


def test_the_cases_walk():
    """For every number of chunks and either tile a walk of several groups, the last one ragged, beyond one chunk with a residual;
    walks of all groups and of a part of them."""
    walks = [(cin, blocks, residual, steps < -(-cout // 256)) for b, h, w, cin, cout, stride, _, _, _, residual, _ in CASES if cout % 256
             for blocks in (2, 4) for steps in [walk(b * -(-h // stride) * -(-w // stride), cout, blocks)] if steps > 1]
    for blocks in (2, 4):
        assert {c for c, k, _, _ in walks if k == blocks} == {64, 128, 192, 256}
        assert {c for c, k, r, _ in walks if k == blocks and r} == {128, 192, 256}
    assert {part for *_, part in walks} == {False, True}


@pytest.mark.parametrize("b,h,w,cin,cout,stride,n,m,tile,residual,bias", CASES)
def test_bits_of_the_strip_form(b, h, w, cin, cout, stride, n, m, tile, residual, bias):
    import torch
    wp = nm.nm_prune(np.random.default_rng(5).standard_normal((cout, 1, 1, cin), dtype=np.float32) * np.float32(0.1), n, m, tile, nm.NM_BF16)
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    x = torch.randn((b, h, w, cin), generator=g, device="cuda").bfloat16()
    ho, wo = -(-h // stride), -(-w // stride)
    res = torch.randn((b, ho, wo, cout), generator=g, device="cuda").bfloat16() if residual else None
    bd = torch.randn(cout, generator=g, device="cuda") if bias else None
    names = {nm.nm_variant_name(v): v for v in range(nm.nm_variant_count())}
    forms = [f for f in names if "_COLS_" in f]
    try:
        for relu in (False, True):
            nm.nm_force_variant(names["SP1_NB4_WP1_NJ2_CK64"])
            ref = nm.nm_conv2d_res(x, wp, res, bd, stride, 0, 1, relu)
            ran = 0
            for f in forms:
                nm.nm_force_variant(names[f])
                say(f"{b}x{h}x{w} {cin} -> {cout} {f}")
                if not f.endswith(f"_C{cin // 64}"):
                    with pytest.raises(nm.NMError) as e:
                        nm.nm_conv2d_res(x, wp, res, bd, stride, 0, 1, relu)
                    assert e.value.code == nm.NM_ERR_UNSUPPORTED
                    continue
                assert torch.equal(nm.nm_conv2d_res(x, wp, res, bd, stride, 0, 1, relu), ref), f
                ran += 1
            assert ran == 2
    finally:
        nm.nm_force_variant(-1)


@pytest.mark.parametrize("b,cin,cout,n,m,pad,cols", [(64, 256, 1024, 2, 4, 0, True), (32, 128, 512, 1, 4, 0, True), (64, 256, 256, 2, 4, 0, False),
                                                     (200, 128, 512, 2, 4, 0, False), (64, 256, 1024, 4, 8, 0, False), (64, 256, 1024, 2, 4, 1, False)])
def test_untuned(b, cin, cout, n, m, pad, cols):
    """14x14 layers on either side of the rule for calls without tuning, against the strip form."""
    import torch
    wp = nm.nm_prune(np.random.default_rng(6).standard_normal((cout, 1, 1, cin), dtype=np.float32) * np.float32(0.1), n, m, 16, nm.NM_BF16)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.rand((b, 14, 14, cin), generator=g, device="cuda").bfloat16()
    say(f"untuned {b} {cin} -> {cout} {n}:{m} pad {pad}")
    y = nm.nm_conv2d(x, wp, None, 1, pad, 1, True)
    assert ("_COLS_" in nm.nm_variant_name(nm.nm_last_variant())) == cols
    names = {nm.nm_variant_name(v): v for v in range(nm.nm_variant_count())}
    try:
        nm.nm_force_variant(names["SP1_NB4_WP1_NJ2_CK64" if n <= 2 else "SP0_NB4_WP1_NJ2_CK64"])
        assert torch.equal(nm.nm_conv2d(x, wp, None, 1, pad, 1, True), y)
    finally:
        nm.nm_force_variant(-1)
