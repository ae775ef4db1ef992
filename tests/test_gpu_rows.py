"""Few input channels out of staged rows (variants RUN_ROWS and ROWF): every form forced on images whose rows, columns and
output heights end inside a workgroup, both alignments of a run, against the CPU oracle."""
import numpy as np
import pytest

from paper_2507_17301_amd import binding as nm
from paper_2507_17301_amd import workloads as wl
from gpu_util import FP32_TOL, BF16_TOL, say, norm_err, oracle_conv

pytestmark = pytest.mark.gpu

L = wl.ConvLayer

# H, W, Cin, Cout, Kh, Kw, stride, pad, dil: even and odd heights, rows of x on and off 16 bytes, a lead-in element or
# none, one to four k-steps, output channels that end inside 64, one output pixel
GRID = [
    (L("stem", 30, 32, 3, 64, 7, 7, 2, 3, 1, 1, 1, 16), 2),
    (L("stem_odd", 29, 26, 3, 64, 7, 7, 2, 3, 1, 1, 1, 16), 3),
    (L("one_pixel", 7, 8, 3, 16, 7, 7, 2, 0, 1, 1, 1, 16), 1),
    (L("cin1", 13, 18, 1, 40, 5, 5, 2, 2, 1, 1, 1, 8), 2),
    (L("cin2_s1", 9, 37, 2, 136, 3, 3, 1, 1, 1, 1, 1, 16), 2),
    (L("cin3_3x3_pruned", 17, 34, 3, 72, 3, 3, 2, 1, 1, 1, 3, 16), 1),
    (L("cin5_wide", 11, 16, 5, 64, 6, 5, 2, 1, 1, 1, 1, 16), 1),
    (L("four_ksteps", 12, 20, 3, 24, 7, 9, 2, 3, 1, 1, 1, 16), 1),
    (L("cin6_T5", 9, 10, 6, 48, 3, 3, 1, 1, 1, 1, 2, 5), 2),
]


def expected_forms(layer, bf16):
    """Names of the forms that this layer's rows, alignment and k-steps ask for (all of GRID's rows fit the LDS)."""
    if (layer.W * layer.Cin) % 2 or (layer.stride * layer.Cin) % 2 or layer.dil != 1:
        return set()
    if layer.Cin % (8 if bf16 else 4) == 0 or layer.Cout % (8 if bf16 else 4):
        return set()
    ks = (layer.Kh * (((layer.pad * layer.Cin) % 2 + layer.Kw * layer.Cin + 7) // 8) + 7) // 8
    if bf16:
        return {f"RUN_ROWS{r}_NJ4_KS{ks}" for r in (1, 2, 4, 8)}
    return {f"ROWF_R{r}_NJ{nj}_KS{ks}" for r in (1, 2, 4, 8) for nj in (1, 2) if ks < 4 or nj == 1}


def each_form(layer, wp, bf16, call):
    """call(name) under each row-staged form in turn: all that are due run, and what else the handle has tables for (the
    k-steps of the other alignment) is refused as a form that cannot run this layer."""
    due, dt = expected_forms(layer, bf16), nm.NM_BF16 if bf16 else nm.NM_F32
    ran = set()
    try:
        for v in range(nm.nm_variant_count()):
            name = nm.nm_variant_name(v)
            if not name.startswith(("RUN_ROWS", "ROWF")) or not nm.nm_variant_legal(v, wp, dt, dt):
                continue
            say(f"{layer.name} {name}")
            nm.nm_force_variant(v)
            if name not in due:
                with pytest.raises(nm.NMError, match="cannot run this layer"):
                    call(name)
                continue
            call(name)
            ran.add(name)
    finally:
        nm.nm_force_variant(-1)
    assert ran == due
    return ran


@pytest.mark.parametrize("layer,batch", GRID, ids=[g[0].name for g in GRID])
@pytest.mark.parametrize("bf16", [False, True], ids=["f32", "bf16"])
def test_every_form(layer, batch, bf16):
    import torch
    x, w, bias = wl.make_tensors(layer, batch, 51, weight_sigma=0.1)
    dt, tdt = (nm.NM_BF16, torch.bfloat16) if bf16 else (nm.NM_F32, torch.float32)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile, dt)
    xd, bd = torch.from_numpy(x).cuda().to(tdt), torch.from_numpy(bias).cuda()
    ref = oracle_conv(layer, x, w, bias, relu=False, bf16=bf16)
    res = torch.from_numpy(np.random.default_rng(5).standard_normal(ref.shape, dtype=np.float32)).cuda().to(tdt)
    tol = BF16_TOL if bf16 else FP32_TOL

    def check(name):
        y = nm.nm_conv2d_res(xd, wp, None, bd, layer.stride, layer.pad, layer.dil, True)
        z = nm.nm_conv2d_res(xd, wp, res, None, layer.stride, layer.pad, layer.dil, False)
        torch.cuda.synchronize()
        assert norm_err(y.float().cpu().numpy(), np.maximum(ref, 0)) <= tol, name
        assert norm_err(z.float().cpu().numpy(), ref - bias + res.float().cpu().numpy()) <= 2 * tol, name   # (ref is rounded too)

    each_form(layer, wp, bf16, check)


def test_infinity_and_default():
    """An infinite pixel reaches exactly the outputs that the element-wise form gives it, and the untuned default runs."""
    import torch
    layer = L("stem", 30, 32, 3, 64, 7, 7, 2, 3, 1, 1, 1, 16)
    x, w, bias = wl.make_tensors(layer, 2, 53)
    x[0, 10, 10, 1], x[1, 0, 0, 2] = np.inf, 1e-38
    wp = nm.nm_prune(w, 1, 1, 16)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    y = nm.nm_conv2d(xd, wp, bd, 2, 3, 1, False)
    assert nm.nm_variant_name(nm.nm_last_variant()).startswith("ROWF")
    base = next(v for v in range(nm.nm_variant_count()) if nm.nm_variant_name(v).startswith("NB4_WP1_NJ1") and nm.nm_variant_legal(v, wp))
    nm.nm_force_variant(base)
    try:
        ref = nm.nm_conv2d(xd, wp, bd, 2, 3, 1, False)
        torch.cuda.synchronize()
    finally:
        nm.nm_force_variant(-1)
    y, ref = y.cpu().numpy(), ref.cpu().numpy()
    fin = np.isfinite(ref)
    # (a run's padding slots are read with weight 0: next to the infinity they may turn a finite sum into NaN, and such
    #  a sum is computed again without them)
    assert (np.isinf(y) == np.isinf(ref)).all() and (np.isnan(y) == np.isnan(ref)).all()
    assert norm_err(y[fin], ref[fin]) <= FP32_TOL


@pytest.mark.parametrize("layer", [GRID[0][0], GRID[3][0], GRID[5][0], GRID[6][0]], ids=lambda l: l.name)
@pytest.mark.parametrize("relu", [False, True])
def test_infinities_bf16(layer, relu):
    """An infinite or NaN pixel reaches the outputs whose window holds it and no other: not those that read it in a padding
    slot (beside the window, or a slot beyond the last kernel row, which reads the window's first pixels)."""
    import torch
    dense = L(layer.name, layer.H, layer.W, layer.Cin, layer.Cout, layer.Kh, layer.Kw, layer.stride, layer.pad, 1, 1, 1, 16)
    x, w, bias = wl.make_tensors(dense, 3, 57, weight_sigma=0.1)
    h, wd, c = dense.H // 2, dense.W // 2, dense.Cin - 1
    x[0, h, wd, 0], x[0, 0, 0, c], x[1, h, wd, c], x[1, dense.H - 1, dense.W - 1, 0] = np.inf, -np.inf, -np.inf, np.nan
    wp = nm.nm_prune(w, 1, 1, 16, nm.NM_BF16)
    xd, bd = torch.from_numpy(x).cuda().to(torch.bfloat16), torch.from_numpy(bias).cuda()
    ref = oracle_conv(dense, np.where(np.isfinite(x), x, 0).astype(np.float32), w, bias, relu=False, bf16=True)
    # where an infinity or NaN arrives, and as what: the same convolution of its sign (a window holds at most one sign)
    mark = np.where(np.isfinite(x), 0, 1).astype(np.float64)
    wt = torch.from_numpy(w).double().permute(0, 3, 1, 2)
    conv = lambda a, k: torch.nn.functional.conv2d(torch.from_numpy(a).permute(0, 3, 1, 2), k, None, dense.stride,
                                                   dense.pad).permute(0, 2, 3, 1).numpy()
    hit = conv(mark, torch.ones_like(wt))
    pos, neg = np.isposinf(x).astype(np.float64), np.isneginf(x).astype(np.float64)
    up = conv(pos, (wt > 0).double()) + conv(neg, (wt < 0).double())
    down = conv(pos, (wt < 0).double()) + conv(neg, (wt > 0).double())
    nan = (conv(np.isnan(x).astype(np.float64), torch.ones_like(wt)) > 0) | ((up > 0) & (down > 0))
    assert (up > 0).any() and (down > 0).any() and nan.any() and (hit == 0).any()

    def check(name):
        y = nm.nm_conv2d(xd, wp, bd, dense.stride, dense.pad, 1, relu)
        torch.cuda.synchronize()
        y = y.float().cpu().numpy()
        ok = hit == 0
        assert norm_err(y[ok], np.maximum(ref, 0)[ok] if relu else ref[ok]) <= BF16_TOL, name
        assert np.isposinf(y[(up > 0) & ~nan]).all(), name
        if relu:
            assert (y[(down > 0) & ~nan] == 0).all(), name
        else:
            assert np.isneginf(y[(down > 0) & ~nan]).all() and np.isnan(y[nan]).all(), name

    assert each_form(dense, wp, True, check)


@pytest.mark.parametrize("layer", [GRID[0][0], GRID[3][0], GRID[5][0]], ids=lambda l: l.name)
@pytest.mark.parametrize("xe,we", [(-118, 40), (-126, 100), (-142, 12), (40, -118)])
def test_values_too_small_for_their_planes(layer, xe, we):
    """fp32: activations whose lower bits lie under bf16's smallest subnormal are computed again; a layer with such
    weights has no row-staged form."""
    import torch
    dense = L(layer.name, layer.H, layer.W, layer.Cin, layer.Cout, layer.Kh, layer.Kw, layer.stride, layer.pad, 1, 1, 1, 16)
    x, w, bias = wl.make_tensors(dense, 2, 59)
    x = np.ldexp(np.random.default_rng(9).standard_normal(x.shape, dtype=np.float32), xe).astype(np.float32)
    w, bias = np.ldexp(w, we).astype(np.float32), bias * 0
    x[:, 3:6] = 0
    wp = nm.nm_prune(w, 1, 1, 16)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2), torch.from_numpy(w).double().permute(0, 3, 1, 2),
                                     None, dense.stride, dense.pad).permute(0, 2, 3, 1).numpy()

    def err(y):
        torch.cuda.synchronize()
        d = y.cpu().numpy().astype(np.float64) - ref
        return float(np.sqrt((d * d).sum() / (ref * ref).sum()))

    legal = [v for v in range(nm.nm_variant_count()) if nm.nm_variant_legal(v, wp)]
    try:
        nm.nm_force_variant(next(v for v in legal if nm.nm_variant_name(v).startswith("NB4_WP1_NJ1")))
        old = err(nm.nm_conv2d(xd, wp, bd, dense.stride, dense.pad, 1, False))
    finally:
        nm.nm_force_variant(-1)

    def check(name):
        e = err(nm.nm_conv2d(xd, wp, bd, dense.stride, dense.pad, 1, False))
        say(f"2^{xe} * 2^{we} {e:.3g} (fp32 instruction {old:.3g})")
        # one rounding per kept column, where the fp32 instruction has one per four: at most twice its distance
        assert e <= 2 * old + 1e-7, name

    if we > -100:
        assert each_form(dense, wp, False, check)
    else:
        assert not any(nm.nm_variant_name(v).startswith("ROWF") for v in legal)
    assert err(nm.nm_conv2d(xd, wp, bd, dense.stride, dense.pad, 1, False)) <= 2 * old + 1e-7


def dist64(y, x, w, bias, layer):
    import torch
    torch.cuda.synchronize()
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2), torch.from_numpy(w).double().permute(0, 3, 1, 2),
                                     torch.from_numpy(bias).double(), layer.stride, layer.pad).permute(0, 2, 3, 1).numpy()
    d = y.cpu().numpy().astype(np.float64) - ref
    return float(np.sqrt((d * d).sum() / (ref * ref).sum()))


@pytest.mark.parametrize("kh,kw,cin,pad", [(1, 1, 7, 0), (3, 3, 1, 1), (1, 9, 1, 0), (2, 2, 2, 0), (1, 1, 10, 0), (4, 4, 1, 1),
                                           (7, 3, 1, 0), (3, 3, 3, 1), (5, 5, 2, 1), (7, 3, 3, 1), (7, 7, 3, 3)])
@pytest.mark.parametrize("kind", ["uniform", "signed"])
@pytest.mark.parametrize("bias_on", [False, True])
def test_no_further_from_float64_than_the_fp32_instruction(kh, kw, cin, pad, kind, bias_on):
    """fp32, also where the kernel's columns are spread thinly over its instructions."""
    import torch
    layer = L("few", 30, 24, cin, 64, kh, kw, 2 if cin % 2 else 1, pad, 1, 1, 1, 16)
    x, w, bias = wl.make_tensors(layer, 4, 61)
    if kind == "signed":
        x = np.random.default_rng(3).standard_normal(x.shape, dtype=np.float32)
    bias = bias * np.float32(bias_on)
    wp = nm.nm_prune(w, 1, 1, 16)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    legal = [v for v in range(nm.nm_variant_count()) if nm.nm_variant_legal(v, wp)]
    run = lambda: nm.nm_conv2d(xd, wp, bd, layer.stride, layer.pad, 1, False)
    try:
        nm.nm_force_variant(next(v for v in legal if nm.nm_variant_name(v).startswith("NB4_WP1_NJ1")))
        old = dist64(run(), x, w, bias, layer)
    finally:
        nm.nm_force_variant(-1)

    def check(name):
        assert dist64(run(), x, w, bias, layer) <= old, name

    assert each_form(layer, wp, False, check)


def test_fewest_columns_keep_the_fp32_instruction():
    """Up to six kept columns the planes' missing products weigh more than the roundings they save."""
    import torch
    for kh, kw, cin in [(1, 1, 1), (1, 3, 1), (2, 2, 1), (1, 1, 5), (1, 3, 2), (1, 1, 6)]:
        layer = L("fewest", 30, 24, cin, 64, kh, kw, 2 if cin % 2 else 1, 0, 1, 1, 1, 16)
        x, w, bias = wl.make_tensors(layer, 2, 63)
        wp = nm.nm_prune(w, 1, 1, 16)
        xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
        say(f"fewest {kh}x{kw}x{cin}")
        nm.nm_conv2d(xd, wp, bd, layer.stride, 0, 1, False)
        assert not nm.nm_variant_name(nm.nm_last_variant()).startswith("ROWF")
        v, _ = nm.nm_autotune(nm.NM_F32, 2, layer.H, layer.W, cin, wp, True, layer.stride, 0, 1, False)
        assert not nm.nm_variant_name(v).startswith("ROWF")
    nm.nm_cache_clear()
