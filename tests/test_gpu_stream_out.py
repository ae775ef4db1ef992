"""Outputs larger than the last-level cache leave through other stores than smaller ones (first layers in bf16 in three ways): a batch on
the far side of a line against its two halves on the near side, bit for bit (the sums of a pixel do not know of the batch)."""
import numpy as np
import pytest

from paper_2507_17301_amd import binding as nm
from gpu_util import say

pytestmark = pytest.mark.gpu

# Every end of a tile that stores in either way: the tile in LDS with 256 and 512 threads (gather, strip and tap-staged forms), the
# row-staged, three-plane, fp8 and channel-walking ones.
CASES = [  # dtype, batch, size, Cin, Cout, k, stride, pad, N:M, residual, variants by prefix ("" = the default)
    ("bf16", 98, 56, 64, 256, 1, 1, 0, (2, 4), True, ("", "SPR1_NB8_WP1_NJ4_CK64", "B16_NB4_WP1_NJ2_SH1")),
    ("bf16", 50, 80, 64, 256, 3, 1, 1, (2, 4), False, ("SPR1_TAPS_NB7_WP2_NJ4",)),
    ("f32", 50, 56, 64, 256, 1, 1, 0, (2, 4), True, ("X3S_NB4_WP1_NJ2", "NB4_WP1_NJ2_CK32")),
    ("bf16", 200, 28, 64, 512, 3, 1, 1, (2, 4), True, ("SPR1_TAP8_NB7_WP2_NJ4", "SPR1_TAP8_NB8_WP2_NJ4")),
    ("bf16", 200, 28, 64, 512, 3, 1, 1, (4, 8), False, ("SPR0_TAP8_NB7_WP2_NJ4", "SPR0_TAP8_NB7_WP2_NJ2")),
    ("bf16", 200, 28, 128, 512, 1, 1, 0, (2, 4), True, ("SPR1_COLS_NB4_C2", "SPR1_COLS_NB2_C2")),
    ("bf16", 200, 28, 256, 512, 1, 1, 0, (2, 4), False, ("", "SPR1_COLS_NB4_C4")),
    ("f32", 100, 28, 64, 512, 3, 1, 1, (2, 4), True, ("X3S_TAP_NB4_WP1_NJ4_KG2", "X3S_TAP_NB4_WP1_NJ4_KG4")),
    ("f32", 100, 28, 64, 512, 3, 1, 1, (4, 8), False, ("X3D_TAP_NB4_WP1_NJ2_KG2", "X3D_TAP_NB4_WP1_NJ2_KG4")),
    ("bf16", 96, 224, 3, 64, 7, 2, 3, (1, 1), False, ("RUN_NB4_WP1_NJ1",)),
    ("bf16", 162, 224, 3, 64, 7, 2, 3, (1, 1), False, ("", "RUN_ROWS4_NJ4")),
    ("bf16", 48, 224, 3, 64, 7, 2, 3, (1, 1), True, ("", "RUN_ROWS1_NJ4", "RUN_ROWS8_NJ4")),
    ("f32", 81, 224, 3, 64, 7, 2, 3, (1, 1), False, ("ROWF_R4_NJ2",)),
    ("f8", 98, 56, 64, 256, 1, 1, 0, (2, 4), False, ("", "F8_NB4_WP1_NJ4")),
]


@pytest.mark.parametrize("dtype,batch,size,cin,cout,k,stride,pad,nm_,residual,variants", CASES)
def test_both_sides_of_the_line(dtype, batch, size, cin, cout, k, stride, pad, nm_, residual, variants):
    import torch
    code, tdt = {"f32": (nm.NM_F32, torch.float32), "bf16": (nm.NM_BF16, torch.bfloat16),
                 "f8": (nm.NM_F8E4M3, torch.float8_e4m3fn)}[dtype]
    rng = np.random.default_rng(17)
    wp = nm.nm_prune(rng.standard_normal((cout, k, k, cin), dtype=np.float32) * np.float32(0.05), *nm_, 16, code)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    x = torch.rand((batch, size, size, cin), generator=g, device="cuda").to(tdt)
    ho = (size + 2 * pad - k) // stride + 1
    ydt = torch.float32 if dtype == "f32" else torch.bfloat16
    res = torch.rand((batch, ho, ho, cout), generator=g, device="cuda").to(ydt) if residual else None
    bias = torch.rand(cout, generator=g, device="cuda")
    half = batch // 2
    yb = batch * ho * ho * cout * (4 if dtype == "f32" else 2)
    lines = {"RUN_NB4_WP1_NJ1": (150e6,), "": (72e6, 256e6)}[variants[0]] if cin == 3 and dtype == "bf16" else (256e6 if cin == 3 else 150e6,)
    assert any(yb * (batch - half) / batch < line < yb for line in lines)
    names = [nm.nm_variant_name(v) for v in range(nm.nm_variant_count())]
    try:
        for want in variants:
            picks = [i for i, n in enumerate(names) if want and n.startswith(want) and nm.nm_variant_legal(i, wp, code, nm.NM_F32 if dtype == "f32" else nm.NM_BF16)]
            picks += [i for i, n in enumerate(names) if n == want and ("_TAP" in n or "_COLS_" in n)]   # (whether these run is decided by the call)
            assert picks or not want, want
            nm.nm_force_variant(picks[0] if want else -1)
            say(f"stream out {dtype} {batch}x{size}x{size}x{cin} -> {cout} {want}")
            y = nm.nm_conv2d_res(x, wp, res, bias, stride, pad, 1, True)
            nm.nm_force_variant(nm.nm_last_variant())
            for lo, hi in ((0, half), (half, batch)):
                part = nm.nm_conv2d_res(x[lo:hi].contiguous(), wp, None if res is None else res[lo:hi].contiguous(), bias, stride, pad, 1, True)
                assert torch.equal(part, y[lo:hi]), (want, lo)
            torch.cuda.synchronize()
            nm.nm_force_variant(-1)
    finally:
        nm.nm_force_variant(-1)
