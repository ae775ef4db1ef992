"""The three-plane fp32 kernel that stages and cuts a tile's input once for all its taps, every form forced: against the CPU oracle
at the edges of its tiles, stages and rounds of chunks, against float64, and with values that planes do not carry."""
import numpy as np
import pytest

from paper_2507_17301_amd import binding as nm
from paper_2507_17301_amd import workloads as wl
from gpu_util import FP32_TOL, norm_err, say
import oracle

pytestmark = pytest.mark.gpu

L = wl.ConvLayer


def forms(sparse):
    return {n: v for v, n in ((v, nm.nm_variant_name(v)) for v in range(nm.nm_variant_count())) if n.startswith("X3S_TAP" if sparse else "X3D_TAP")}


def run(v, x, wp, b, pad, dil, relu, res=None):
    import torch
    nm.nm_force_variant(v)
    try:
        y = nm.nm_conv2d_res(x, wp, res, b, 1, pad, dil, relu)
        torch.cuda.synchronize()
        return y.cpu().numpy()
    finally:
        nm.nm_force_variant(-1)


def fp32_instruction(wp):
    return next(v for v in range(nm.nm_variant_count()) if nm.nm_variant_name(v).startswith("NB4_WP1_NJ1") and nm.nm_variant_legal(v, wp))


def conv64(x, wz, bias):
    import torch
    y = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2), torch.from_numpy(wz).double().permute(0, 3, 1, 2),
                                   torch.from_numpy(bias).double(), 1, 1)
    return y.permute(0, 2, 3, 1).numpy()


def rel64(got, ref):
    d = got.astype(np.float64) - ref
    return float(np.sqrt((d * d).sum() / (ref * ref).sum()))


# H, W, Cin, Cout, kernel, dilation, n, m, tile, batch: a pixel; one to five stages; fewer, as many and more taps than groups,
# rounds with chunks left over (nine taps of one stage, 15 chunks); outputs that are no whole quads, row blocks or tiles
GRID = [(1, 1, 64, 16, (3, 3), (1, 1), 2, 4, 16, 1), (9, 13, 64, 37, (3, 3), (1, 1), 1, 4, 5, 2), (14, 14, 256, 264, (3, 3), (1, 1), 2, 4, 16, 3),
        (7, 7, 320, 128, (3, 3), (1, 1), 2, 8, 8, 5), (11, 10, 192, 72, (1, 3), (1, 2), 2, 4, 16, 3), (12, 9, 128, 136, (2, 2), (2, 2), 2, 4, 32, 2),
        (6, 7, 64, 64, (5, 5), (1, 1), 2, 4, 16, 3), (5, 12, 192, 40, (5, 1), (1, 1), 2, 4, 16, 2),
        (14, 13, 128, 130, (3, 3), (1, 1), 64, 128, 16, 2), (8, 8, 64, 72, (3, 3), (2, 2), 1, 1, 16, 3), (7, 7, 192, 100, (3, 3), (1, 1), 4, 8, 4, 4)]
# one stage of more granules than the threads hold at a time (three each): two to three passes over it, the last one ragged
WIDE = [(56, 56, 64, 130, (3, 3), (1, 1), 2, 4, 16, 2), (28, 100, 64, 72, (3, 3), (1, 1), 1, 4, 8, 2), (30, 40, 64, 40, (5, 5), (1, 1), 2, 4, 16, 2),
        (40, 44, 64, 36, (3, 3), (1, 1), 1, 1, 16, 2), (30, 90, 64, 72, (3, 3), (1, 1), 4, 8, 16, 1)]


def granules(h, w, ph, pw, pixels=64):
    """16-byte granules that a tile of 64 pixels and what its taps reach span at most: nine a pixel, and the zeros between rows and images."""
    line = 9 * w + (9 * pw + 7) // 8 * 8
    return 9 * pixels + (pixels + w - 2) // w * (line - 9 * w) + (pixels + h * w - 2) // (h * w) * ph * line + 2 * (ph * line + 9 * pw)


def test_the_wide_layers_are_wide():
    for h, w, cin, _, k, dil, *_ in WIDE:
        assert cin == 64 and granules(h, w, dil[0] * (k[0] - 1) // 2, dil[1] * (k[1] - 1) // 2) > 3 * 512


@pytest.mark.parametrize("h,w,cin,cout,k,dil,n,m,tile,batch", GRID + WIDE)
def test_every_form(h, w, cin, cout, k, dil, n, m, tile, batch):
    import torch
    rng = np.random.default_rng(11)
    wt = rng.standard_normal((cout, *k, cin), dtype=np.float32) * np.float32((2 / (k[0] * k[1] * cin)) ** 0.5)
    x, bias = rng.standard_normal((batch, h, w, cin), dtype=np.float32), rng.standard_normal(cout, dtype=np.float32)
    res = rng.standard_normal((batch, h, w, cout), dtype=np.float32)
    pad = (dil[0] * (k[0] - 1) // 2, dil[1] * (k[1] - 1) // 2)
    ref = oracle.conv2d(x, oracle.prune(wt, n, m, tile)[2], bias, 1, pad, dil, False)
    wp = nm.nm_prune(wt, n, m, tile)
    xd, bd, rd = (torch.from_numpy(a).cuda() for a in (x, bias, res))
    sparse = n <= 2 and m % 4 == 0
    ran = 0
    for name, v in forms(sparse).items():
        assert not nm.nm_variant_legal(v, wp)   # depends on more than the handle
        say(f"{h}x{w} {cin}->{cout} {k} {name}")
        if k[0] * k[1] < int(name[-1]):
            with pytest.raises(nm.NMError) as e:
                run(v, xd, wp, bd, pad, dil, True)
            assert e.value.code == nm.NM_ERR_UNSUPPORTED
            continue
        assert norm_err(run(v, xd, wp, bd, pad, dil, True), np.maximum(ref, 0)) <= FP32_TOL, name
        assert norm_err(run(v, xd, wp, bd, pad, dil, False, rd), ref + res) <= FP32_TOL, name
        assert norm_err(run(v, xd, wp, None, pad, dil, False), ref - bias) <= FP32_TOL, name
        ran += 1
    assert ran


@pytest.mark.parametrize("h,w,cin,k,n,m", [(7, 7, 64, (3, 3), 2, 4), (5, 6, 128, (3, 3), 1, 1), (7, 9, 192, (3, 5), 2, 4), (6, 7, 64, (5, 1), 4, 8),
                                           (14, 14, 320, (3, 3), 1, 4)])
def test_an_image_gives_the_same_bits_wherever_it_is_in_the_batch(h, w, cin, k, n, m):
    """Images that begin at every place of a tile, with chunks left over beyond whole rounds of the groups (9, 18, 45, 5 and 45 chunks)."""
    import torch
    rng = np.random.default_rng(3)
    wp = nm.nm_prune(rng.standard_normal((72, *k, cin), dtype=np.float32) * np.float32(0.1), n, m, 16)
    one = torch.from_numpy(rng.standard_normal((1, h, w, cin), dtype=np.float32)).cuda()
    x = one.expand(19, h, w, cin).contiguous()
    pad = ((k[0] - 1) // 2, (k[1] - 1) // 2)
    bias = torch.from_numpy(rng.standard_normal(72, dtype=np.float32)).cuda()
    for name, v in forms(n <= 2 and m % 4 == 0).items():
        say(f"place in the batch {h}x{w} {cin} {k} {name}")
        y = run(v, x, wp, bias, pad, (1, 1), False)
        assert (y == y[:1]).all() and (y[:1] == run(v, one, wp, bias, pad, (1, 1), False)).all(), name


@pytest.mark.parametrize("n,m,cin", [(2, 4, 64), (2, 4, 512), (1, 1, 64), (4, 8, 256)])
@pytest.mark.parametrize("kind", ["uniform", "signed", "tiny"])
def test_no_further_from_float64_than_the_fp32_instruction(n, m, cin, kind):
    import torch
    layer = L("acc", 14, 14, cin, 64, 3, 3, 1, 1, 1, n, m, 16)
    x, w, bias = wl.make_tensors(layer, 2, 17)
    if kind != "uniform":
        x = np.random.default_rng(3).standard_normal(x.shape, dtype=np.float32)
    if kind == "tiny":                          # the third planes are subnormal
        x, bias = x * np.float32(1e-33), bias * 0
    wp = nm.nm_prune(w, n, m, 16)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = conv64(x, oracle.prune(w, n, m, 16)[2], bias)
    old = rel64(run(fp32_instruction(wp), xd, wp, bd, 1, 1, False), ref)
    for name, v in forms(n <= 2 and m % 4 == 0).items():
        e = rel64(run(v, xd, wp, bd, 1, 1, False), ref)
        say(f"{n}:{m} {cin} {kind} {name} {e:.3g} (fp32 instruction {old:.3g})")
        assert e <= old, name


@pytest.mark.parametrize("tile,cout", [(1, 20), (4, 36), (16, 37), (16, 136), (32, 72)])
@pytest.mark.parametrize("n,m", [(2, 4), (1, 1)])
def test_infinities_and_values_too_small_for_planes(tile, cout, n, m):
    """Outputs that are computed again, singly or four channels at a time, with residual and ReLU: image 0 holds activations whose
    lower bits lie under bf16's smallest subnormal, lifted by the weights, image 1 infinities, a NaN and the largest numbers."""
    import torch
    layer = L("again", 11, 10, 128, cout, 3, 3, 1, 1, 1, n, m, tile)
    x, w, bias = wl.make_tensors(layer, 2, 43)
    x[0], bias = np.ldexp(x[0] - 0.5, -118), bias * 0
    x[1, 4, 5, 7], x[1, 9, 0, 60], x[1, 0, 9, 100], x[1, 10, 5, 1] = np.inf, -np.inf, np.nan, 3.4e38
    w = np.ldexp(w, 30).astype(np.float32)
    wp = nm.nm_prune(w, n, m, tile)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    for relu in (False, True):
        ref = run(fp32_instruction(wp), xd, wp, bd, 1, 1, relu)
        rd = torch.from_numpy(np.random.default_rng(3).standard_normal(ref.shape, dtype=np.float32)).cuda()
        ref2 = run(fp32_instruction(wp), xd, wp, bd, 1, 1, relu, rd)
        ok = np.isfinite(ref)
        assert ok[0].all() and not ok[1].all()
        for name, v in forms(n <= 2 and m % 4 == 0).items():
            say(f"again {n}:{m} T{tile} {cout} {relu} {name}")
            got = run(v, xd, wp, bd, 1, 1, relu)
            assert rel64(got[0], ref[0].astype(np.float64)) <= 1e-6, name
            assert (np.isnan(got) == np.isnan(ref)).all() and (got[np.isinf(ref)] == ref[np.isinf(ref)]).all(), name
            assert rel64(got[ok], ref[ok].astype(np.float64)) <= 1e-6, name
            got = run(v, xd, wp, bd, 1, 1, relu, rd)
            assert rel64(got[0], ref2[0].astype(np.float64)) <= 1e-6, name


@pytest.mark.parametrize("cin,n,m", [(64, 2, 4), (192, 2, 4), (64, 1, 1), (192, 4, 8)])
@pytest.mark.parametrize("xe,we", [(-118, 40), (-126, 100), (-142, 12), (-95, 0)])
def test_activations_too_small_for_their_planes(cin, n, m, xe, we):
    """In one stage only, the last one of three too: as near to float64 as the fp32 instruction."""
    import torch
    layer = L("small", 12, 11, cin, 72, 3, 3, 1, 1, 1, n, m, 16)
    x, w, bias = wl.make_tensors(layer, 2, 23)
    x = np.random.default_rng(7).standard_normal(x.shape, dtype=np.float32)
    x[..., :cin - 64] = 0
    x, w, bias = np.ldexp(x, xe).astype(np.float32), np.ldexp(w, we).astype(np.float32), bias * 0
    wp = nm.nm_prune(w, n, m, 16)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = conv64(x, oracle.prune(w, n, m, 16)[2], bias)
    old = rel64(run(fp32_instruction(wp), xd, wp, bd, 1, 1, False), ref)
    for name, v in forms(n <= 2 and m % 4 == 0).items():
        e = rel64(run(v, xd, wp, bd, 1, 1, False), ref)
        say(f"{n}:{m} {cin} 2^{xe} * 2^{we} {name} {e:.3g} (fp32 instruction {old:.3g})")
        # one rounding per kept column, where the fp32 instruction has one per four: at most twice its distance
        assert e <= 2 * old + 1e-7, name


@pytest.mark.parametrize("batch,cin,cout,n,m,form", [(32, 256, 256, 2, 4, "X3S_TAP_"), (64, 256, 256, 2, 4, "X3S_TAP_NB4_WP1_NJ4_KG2"),
                                                     (8, 128, 256, 2, 4, "X3S_NB"), (120, 128, 128, 2, 4, "X3S_NB"),
                                                     (60, 64, 128, 4, 8, "X3D_TAP_"), (120, 128, 128, 1, 1, "X3D_NB")])
def test_untuned(batch, cin, cout, n, m, form):
    """14x14 layers on either side of the rule for calls without tuning, sampled outputs against the oracle."""
    import torch
    layer = L("untuned", 14, 14, cin, cout, 3, 3, 1, 1, 1, n, m, 16)
    x, w, bias = wl.make_tensors(layer, batch, 9)
    wp = nm.nm_prune(w, n, m, 16)
    say(f"untuned {batch} {cin} -> {cout} {n}:{m}")
    y = nm.nm_conv2d(torch.from_numpy(x).cuda(), wp, torch.from_numpy(bias).cuda(), 1, 1, 1, True)
    assert nm.nm_variant_name(nm.nm_last_variant()).startswith(form), nm.nm_variant_name(nm.nm_last_variant())
    pts = wl.sample_points(layer, batch, 2000, 1)
    ref = oracle.conv2d_points(x, oracle.prune(w, n, m, 16)[2], pts, bias, 1, 1, 1, True)
    assert norm_err(y.cpu().numpy()[pts[:, 0], pts[:, 1], pts[:, 2], pts[:, 3]], ref) <= FP32_TOL


def test_untuned_wide():
    """56x56: one stage in two passes, as a call without tuning runs it; sampled outputs against the oracle."""
    import torch
    layer = L("wide", 56, 56, 64, 128, 3, 3, 1, 1, 1, 2, 4, 16)
    assert granules(56, 56, 1, 1) > 3 * 512
    x, w, bias = wl.make_tensors(layer, 4, 13)
    wp = nm.nm_prune(w, 2, 4, 16)
    say("untuned 56x56 64 -> 128")
    y = nm.nm_conv2d(torch.from_numpy(x).cuda(), wp, torch.from_numpy(bias).cuda(), 1, 1, 1, True)
    assert nm.nm_variant_name(nm.nm_last_variant()).startswith("X3S_TAP_"), nm.nm_variant_name(nm.nm_last_variant())
    pts = wl.sample_points(layer, 4, 4000, 1)
    ref = oracle.conv2d_points(x, oracle.prune(w, 2, 4, 16)[2], pts, bias, 1, 1, 1, True)
    assert norm_err(y.cpu().numpy()[pts[:, 0], pts[:, 1], pts[:, 2], pts[:, 3]], ref) <= FP32_TOL
