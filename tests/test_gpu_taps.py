"""The bf16 kernel that stages a tile's input once for all taps, every form forced, against the CPU oracle: edges of its
tiles, of the images and of the stages; the calls that it refuses; and the layers that take it without tuning."""
import numpy as np
import pytest

import oracle
from paper_2507_17301_amd import binding as nm
from paper_2507_17301_amd import workloads as wl
from gpu_util import BF16_TOL, say, norm_err, oracle_conv

pytestmark = pytest.mark.gpu

L = wl.ConvLayer

CASES = [
    # name, H, W, Cin, Cout, Kh, Kw, stride, pad, dil, n, m, tile | batch, residual
    (L("tap_one_pixel", 1, 1, 64, 16, 3, 3, 1, 1, 1, 2, 4, 16), 1, False),     # eight of nine taps outside
    (L("tap_one_stage", 9, 13, 64, 64, 3, 3, 1, 1, 1, 2, 4, 16), 3, False),    # images end inside a tile
    (L("tap_7x7_c72", 7, 7, 128, 72, 3, 3, 1, 1, 1, 2, 8, 16), 10, True),      # many images a tile, channels end inside it
    (L("tap_W1", 65, 1, 128, 24, 3, 3, 1, 1, 1, 1, 4, 16), 2, False),          # a row end after every pixel
    (L("tap_3stages_T32", 14, 14, 192, 160, 3, 3, 1, 1, 1, 4, 8, 32), 2, False),
    (L("tap_4stages", 15, 15, 256, 136, 3, 3, 1, 1, 1, 1, 8, 32), 1, True),
    (L("tap_dil2", 11, 17, 128, 128, 3, 3, 1, 2, 2, 1, 4, 32), 2, True),
    (L("tap_5x5", 10, 6, 64, 40, 5, 5, 1, 2, 1, 2, 4, 16), 3, False),
    (L("tap_448", 16, 28, 64, 64, 3, 3, 1, 1, 1, 2, 4, 16), 1, False),         # exactly one of the largest tiles
    (L("tap_449", 449, 1, 64, 64, 3, 3, 1, 1, 1, 1, 1, 16), 1, False),         # dense, one pixel more
]
REFUSED = [(L("s2", 8, 8, 64, 64, 3, 3, 2, 1, 1, 2, 4, 16)), (L("pad0", 8, 8, 64, 64, 3, 3, 1, 0, 1, 2, 4, 16)),
           (L("pad2", 8, 8, 64, 64, 3, 3, 1, 2, 1, 2, 4, 16)), (L("T8", 8, 8, 64, 64, 3, 3, 1, 1, 1, 2, 4, 8)),
           (L("cout12", 8, 8, 64, 12, 3, 3, 1, 1, 1, 2, 4, 16)), (L("cin96", 8, 8, 96, 64, 3, 3, 1, 1, 1, 2, 4, 16)),
           (L("1x1", 8, 8, 64, 64, 1, 1, 1, 0, 1, 2, 4, 16))]


def _forms():
    return {nm.nm_variant_name(v): v for v in range(nm.nm_variant_count()) if "_TAPS_" in nm.nm_variant_name(v)}


@pytest.mark.parametrize("layer,batch,with_res", CASES, ids=[c[0].name for c in CASES])
def test_every_form(layer, batch, with_res):
    import torch
    x, w, bias = wl.make_tensors(layer, batch, 71)
    x = x * 2 - 1
    ref = oracle_conv(layer, x, w, bias, False, bf16=True)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile, nm.NM_BF16)
    xd, bd = torch.from_numpy(x).cuda().to(torch.bfloat16), torch.from_numpy(bias).cuda()
    rd = None
    if with_res:
        rd = torch.from_numpy(np.random.default_rng(3).standard_normal(ref.shape, dtype=np.float32)).cuda().to(torch.bfloat16)
        ref = oracle.conv2d(oracle.round_bf16(x), oracle.round_bf16(oracle.prune(w, layer.n, layer.m, layer.tile)[2]), bias,
                            layer.stride, layer.pad, layer.dil, False) + rd.float().cpu().numpy()
    ref = np.maximum(ref, 0)
    sparse = layer.n <= 2 and layer.m % 4 == 0
    ran = set()
    try:
        for name, v in _forms().items():
            assert not nm.nm_variant_legal(v, wp, nm.NM_BF16, nm.NM_BF16)   # depends on more than the handle
            say(f"{layer.name} {name}")
            nm.nm_force_variant(v)
            try:
                y = nm.nm_conv2d_res(xd, wp, rd, bd, layer.stride, layer.pad, layer.dil, True)
            except nm.NMError as e:
                assert e.code == nm.NM_ERR_UNSUPPORTED
                continue
            torch.cuda.synchronize()
            assert norm_err(y.float().cpu().numpy(), ref) <= BF16_TOL, name
            ran.add(name)
    finally:
        nm.nm_force_variant(-1)
    # the smaller tiles fit the LDS on all of these
    assert {"SPR0_TAPS_NB5_WP2_NJ4"} <= ran and ("SPR1_TAPS_NB4_WP1_NJ2" in ran) == sparse


@pytest.mark.parametrize("layer", REFUSED, ids=[l.name for l in REFUSED])
def test_refused(layer):
    import torch
    x, w, bias = wl.make_tensors(layer, 1, 5)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile, nm.NM_BF16)
    xd = torch.from_numpy(x).cuda().to(torch.bfloat16)
    try:
        for v in _forms().values():
            nm.nm_force_variant(v)
            with pytest.raises(nm.NMError, match="cannot run this layer"):
                nm.nm_conv2d(xd, wp, None, layer.stride, layer.pad, layer.dil, True)
    finally:
        nm.nm_force_variant(-1)


# one round of 224-pixel tiles, one of 160, several of 448 x 64, 2:8 of a wider tile; too few workgroups; then layers on which the
# form that would otherwise be taken is slower than the strip-per-tap one: half of its 256 channels exist (194 workgroups of
# 160 x 128 are too few), a second round of workgroups that has only begun
@pytest.mark.parametrize("layer,batch,tap", [
    (L("d_28", 28, 28, 128, 128, 3, 3, 1, 1, 1, 2, 4, 16), 64, True), (L("d_odd", 61, 59, 128, 128, 3, 3, 1, 1, 1, 2, 8, 16), 11, True),
    (L("d_56", 56, 56, 64, 64, 3, 3, 1, 1, 1, 2, 4, 16), 32, True), (L("d_T32", 21, 19, 192, 384, 3, 3, 1, 1, 1, 1, 4, 32), 37, True),
    (L("d_small", 14, 14, 256, 256, 3, 3, 1, 1, 1, 2, 4, 16), 4, False),
    (L("d_half", 35, 10, 128, 128, 3, 3, 1, 1, 1, 2, 4, 16), 71, False), (L("d_begun", 32, 52, 64, 64, 3, 3, 1, 1, 1, 1, 4, 16), 80, False)], ids=lambda a: getattr(a, "name", None))
def test_untuned_default(layer, batch, tap):
    import torch
    x, w, bias = wl.make_tensors(layer, batch, 9)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile, nm.NM_BF16)
    xd, bd = torch.from_numpy(x).cuda().to(torch.bfloat16), torch.from_numpy(bias).cuda()
    say(layer.name)
    y = nm.nm_conv2d(xd, wp, bd, layer.stride, layer.pad, layer.dil, True)
    torch.cuda.synchronize()
    assert ("_TAPS_" in nm.nm_variant_name(nm.nm_last_variant())) == tap
    pts = wl.sample_points(layer, batch, 3000, 1)
    ref = oracle_conv(layer, x, w, bias, True, bf16=True, pts=pts)
    got = y.float().cpu().numpy()[pts[:, 0], pts[:, 1], pts[:, 2], pts[:, 3]]
    assert norm_err(got, ref) <= BF16_TOL
