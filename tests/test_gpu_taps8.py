"""The tap-staged bf16 kernel with eight contracting wavefronts adds in the order of the form with four: the same bits, at the edges
of its tiles (a pixel, ragged pixels and channels, several images in a tile), over one to five stages, and with two taps a stage,
where the requests of a stage are only a chunk older than the wait for them."""
import numpy as np
import pytest

from paper_2507_17301_amd import binding as nm
from gpu_util import say

pytestmark = pytest.mark.gpu

CASES = [  # B, H, W, Cin, Cout, kernel, dilation, N, M, T, residual
    (1, 1, 1, 64, 16, (3, 3), (1, 1), 2, 4, 16, False), (1, 9, 13, 64, 40, (3, 3), (1, 1), 1, 4, 16, True),
    (5, 14, 14, 256, 256, (3, 3), (1, 1), 2, 8, 32, False), (7, 7, 7, 320, 264, (3, 3), (1, 1), 4, 8, 16, True),
    (3, 11, 17, 192, 136, (1, 2), (1, 2), 2, 4, 16, False), (2, 16, 14, 128, 512, (2, 2), (2, 2), 2, 4, 16, True),
    (2, 15, 30, 128, 128, (5, 5), (1, 1), 1, 1, 16, False), (16, 14, 14, 128, 248, (3, 3), (2, 2), 2, 4, 16, True),
]


@pytest.mark.parametrize("b,h,w,cin,cout,k,dil,n,m,tile,residual", CASES)
def test_bits_of_the_form_with_four(b, h, w, cin, cout, k, dil, n, m, tile, residual):
    import torch
    rng = np.random.default_rng(5)
    wp = nm.nm_prune(rng.standard_normal((cout, *k, cin), dtype=np.float32) * np.float32(0.05), n, m, tile, nm.NM_BF16)
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    x = torch.randn((b, h, w, cin), generator=g, device="cuda").bfloat16()
    res = torch.randn((b, h, w, cout), generator=g, device="cuda").bfloat16() if residual else None
    bias = torch.randn(cout, generator=g, device="cuda")
    pad = (dil[0] * (k[0] - 1) // 2, dil[1] * (k[1] - 1) // 2)
    forms = {nm.nm_variant_name(v): v for v in range(nm.nm_variant_count()) if "_TAP" in nm.nm_variant_name(v)}
    out = {}
    try:
        for name, v in forms.items():
            nm.nm_force_variant(v)
            say(f"{h}x{w} {cin} -> {cout} {k} {name}")
            try:
                out[name] = nm.nm_conv2d_res(x, wp, res, bias, 1, pad, dil, True)
            except nm.NMError as e:
                assert e.code == nm.NM_ERR_UNSUPPORTED
        torch.cuda.synchronize()
    finally:
        nm.nm_force_variant(-1)
    wide = [f for f in out if "_TAP8_" in f]
    # (a tile of one-pixel images is more rows of zeros than a workgroup's requests cover)
    assert len(wide) == 0 if h * w == 1 else wide
    for f in wide:
        four = [a for a in out if a.startswith(f[:5] + "TAPS_")]
        assert four and torch.equal(out[f], out[four[0]]), f


@pytest.mark.parametrize("b,cin,cout,n,m,form", [(244, 128, 256, 2, 4, "SPR1_TAP8_"), (96, 64, 512, 4, 8, "SPR0_TAP8_"),
                                                 (230, 64, 384, 1, 1, "SPR0_TAP8_"), (20, 64, 256, 4, 8, "SP"),
                                                 (61, 128, 256, 2, 4, "SP")])
def test_untuned(b, cin, cout, n, m, form):
    """14x14 layers on either side of the rule for calls without tuning, against the strip-per-tap form."""
    import torch
    rng = np.random.default_rng(6)
    wp = nm.nm_prune(rng.standard_normal((cout, 3, 3, cin), dtype=np.float32) * np.float32(0.05), n, m, 16, nm.NM_BF16)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    x = torch.rand((b, 14, 14, cin), generator=g, device="cuda").bfloat16()
    say(f"untuned {b} {cin} -> {cout}")
    y = nm.nm_conv2d(x, wp, None, 1, 1, 1, False)
    name = nm.nm_variant_name(nm.nm_last_variant())
    assert name.startswith(form) and ("_TAP8_" in name) == form.endswith("TAP8_"), name
    sparse = int(n <= 2 and m % 4 == 0)
    names = {nm.nm_variant_name(v): v for v in range(nm.nm_variant_count())}
    try:
        nm.nm_force_variant(names[f"SPR{sparse}_NB8_WP1_NJ2_CK64"])
        ref = nm.nm_conv2d(x, wp, None, 1, 1, 1, False)
    finally:
        nm.nm_force_variant(-1)
    # two roundings to bf16 of sums that differ in the last bits of fp32: equal but for the few next to a midpoint
    assert ((y.float() - ref.float()).norm() / ref.float().norm()).item() < 1e-3
