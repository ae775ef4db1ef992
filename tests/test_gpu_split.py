"""fp32 tensors as three bf16 planes (variants X3S / X3D): every form forced on shapes at the edges of
its tiles, against the CPU oracle and, for accuracy and for infinities, against the fp32-instruction form."""
import numpy as np
import pytest

from paper_2507_17301_amd import binding as nm
from paper_2507_17301_amd import workloads as wl
from gpu_util import FP32_TOL, say, norm_err, oracle_conv

pytestmark = pytest.mark.gpu

L = wl.ConvLayer

# H, W, Cin, Cout, Kh, Kw, stride, pad, dil, n, m, tile (+ batch): pixel counts around 32 / 64 / 96 / 128, channel counts
# that end inside a chunk or a row block, one chunk and odd and even numbers of them, column tiles that are no row block
GRID = [
    (L("one_pixel", 3, 3, 64, 16, 3, 3, 1, 0, 1, 2, 4, 16), 1),
    (L("P31_cin4", 31, 1, 4, 9, 1, 1, 1, 0, 1, 2, 4, 16), 1),
    (L("P33_cin68", 11, 3, 68, 36, 1, 1, 1, 0, 1, 1, 4, 8), 1),
    (L("P64_T1", 8, 8, 64, 20, 3, 3, 1, 1, 1, 2, 8, 1), 1),
    (L("P129_T5", 43, 3, 128, 37, 1, 1, 1, 0, 1, 2, 4, 5), 1),
    (L("s2_dil2", 15, 13, 48, 72, 3, 3, 2, 2, 2, 1, 8, 8), 3),
    (L("T32", 10, 10, 192, 144, 1, 1, 1, 0, 1, 2, 4, 32), 2),
    (L("multi", 19, 17, 64, 272, 3, 3, 1, 1, 1, 2, 4, 16), 2),
    (L("dense", 9, 11, 72, 48, 3, 3, 1, 1, 1, 1, 1, 16), 2),
    (L("k4of8", 9, 7, 64, 80, 3, 3, 1, 1, 1, 4, 8, 16), 2),
    (L("cin_groups", 10, 9, 128, 40, 3, 3, 1, 1, 1, 64, 128, 16), 2),
]


def split_variants(wp):
    return [v for v in range(nm.nm_variant_count())
            if nm.nm_variant_name(v).startswith("X3") and nm.nm_variant_legal(v, wp)]


def fp32_instruction(wp):
    return next(v for v in range(nm.nm_variant_count())
                if nm.nm_variant_name(v).startswith("NB4_WP1_NJ1") and nm.nm_variant_legal(v, wp))


def run(v, x, wp, b, layer, relu=True, res=None):
    import torch
    nm.nm_force_variant(v)
    try:
        y = nm.nm_conv2d_res(x, wp, res, b, layer.stride, layer.pad, layer.dil, relu)
        torch.cuda.synchronize()
        assert nm.nm_last_variant() == v
        return y.cpu().numpy()
    finally:
        nm.nm_force_variant(-1)


@pytest.mark.parametrize("layer,batch", GRID, ids=[g[0].name for g in GRID])
def test_every_form(layer, batch):
    import torch
    x, w, bias = wl.make_tensors(layer, batch, 31, weight_sigma=0.1)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = oracle_conv(layer, x, w, bias, relu=False)
    res = np.random.default_rng(5).standard_normal(ref.shape, dtype=np.float32)
    vs = split_variants(wp)
    assert vs
    for v in vs:
        say(f"{layer.name} {nm.nm_variant_name(v)}")
        assert norm_err(run(v, xd, wp, bd, layer, relu=True), np.maximum(ref, 0)) <= FP32_TOL, nm.nm_variant_name(v)
        got = run(v, xd, wp, bd, layer, relu=False, res=torch.from_numpy(res).cuda())
        assert norm_err(got, ref + res) <= FP32_TOL, nm.nm_variant_name(v)


@pytest.mark.parametrize("layer", [L("k18", 20, 20, 36, 64, 1, 1, 1, 0, 1, 2, 4, 16), L("k32", 20, 20, 64, 64, 1, 1, 1, 0, 1, 2, 4, 16),
                                   L("k288", 20, 20, 64, 64, 3, 3, 1, 1, 1, 2, 4, 16),
                                   L("k2304", 14, 14, 512, 64, 3, 3, 1, 1, 1, 2, 4, 16),
                                   L("dense576", 14, 14, 64, 64, 3, 3, 1, 1, 1, 1, 1, 16)], ids=lambda l: l.name)
@pytest.mark.parametrize("kind", ["uniform", "signed", "tiny"])
def test_no_further_from_float64_than_the_fp32_instruction(layer, kind):
    import torch
    x, w, bias = wl.make_tensors(layer, 2, 17)
    if kind != "uniform":
        x = np.random.default_rng(3).standard_normal(x.shape, dtype=np.float32)
    if kind == "tiny":                          # the third planes are subnormal
        x, bias = x * np.float32(1e-33), bias * 0
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    idx = nm.nm_packed_indices(wp).reshape(-1, layer.K // layer.m * layer.n)
    vals = nm.nm_packed_values(wp).reshape(*idx.shape, layer.tile)
    wz = np.zeros((layer.Cout, layer.K))
    for j in range(idx.shape[0]):
        for t in range(layer.tile):
            wz[j * layer.tile + t, idx[j]] = vals[j, :, t]
    wt = torch.from_numpy(wz.reshape(layer.Cout, layer.Kh, layer.Kw, layer.Cin)).permute(0, 3, 1, 2)
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2), wt,
                                     torch.from_numpy(bias).double(), layer.stride, layer.pad, layer.dil)
    ref = ref.permute(0, 2, 3, 1).numpy()

    def err(v):
        d = run(v, xd, wp, bd, layer, relu=False).astype(np.float64) - ref
        return float(np.sqrt((d * d).sum() / (ref * ref).sum()))

    old = err(fp32_instruction(wp))
    for v in split_variants(wp):
        e = err(v)
        say(f"{layer.name} {nm.nm_variant_name(v)} {e:.3g} (fp32 instruction {old:.3g})")
        assert e <= old, nm.nm_variant_name(v)


@pytest.mark.parametrize("relu", [False, True])
def test_infinities_and_nan(relu):
    """Infinite and NaN activations give what the fp32 instruction gives."""
    import torch
    layer = L("inf", 12, 12, 64, 64, 3, 3, 1, 1, 1, 2, 4, 16)
    x, w, bias = wl.make_tensors(layer, 2, 19)
    w[w == 0] = 0.01
    x[0, 2, 3, 5], x[0, 9, 9, 40], x[1, 4, 4, 10] = np.inf, -np.inf, np.nan
    x[1, 9, 9, 3] = 3.4e38                      # next to the largest number; the sums stay finite
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = run(fp32_instruction(wp), xd, wp, bd, layer, relu)
    assert np.isnan(ref).any() or relu
    assert np.isinf(ref).any()
    for v in split_variants(wp):
        say(f"inf {nm.nm_variant_name(v)}")
        got = run(v, xd, wp, bd, layer, relu)
        assert (np.isnan(got) == np.isnan(ref)).all(), nm.nm_variant_name(v)
        same = (got == ref) | ~np.isinf(ref)
        assert same.all() and not np.isinf(got[np.isfinite(ref)]).any(), nm.nm_variant_name(v)
        ok = np.isfinite(ref)
        assert norm_err(got[ok], ref[ok]) <= FP32_TOL


def zero_filled(wp, layer):
    idx = nm.nm_packed_indices(wp).reshape(-1, layer.K // layer.m * layer.n)
    vals = nm.nm_packed_values(wp).reshape(*idx.shape, layer.tile)
    wz = np.zeros((layer.Cout, layer.K))
    for j in range(idx.shape[0]):
        for t in range(layer.tile):
            if j * layer.tile + t < layer.Cout:
                wz[j * layer.tile + t, idx[j]] = vals[j, :, t]
    return wz.reshape(layer.Cout, layer.Kh, layer.Kw, layer.Cin)


def conv64(layer, x, wz, bias):
    import torch
    ref = torch.nn.functional.conv2d(torch.from_numpy(x).double().permute(0, 3, 1, 2), torch.from_numpy(wz).permute(0, 3, 1, 2),
                                     torch.from_numpy(bias).double(), layer.stride, layer.pad, layer.dil)
    return ref.permute(0, 2, 3, 1).numpy()


def rel64(got, ref):
    d = got.astype(np.float64) - ref
    return float(np.sqrt((d * d).sum() / (ref * ref).sum()))


SMALL = [L("sparse", 12, 11, 64, 64, 3, 3, 1, 1, 1, 2, 4, 16), L("dense", 12, 11, 64, 72, 3, 3, 1, 1, 1, 1, 1, 16)]


@pytest.mark.parametrize("layer", SMALL, ids=lambda l: l.name)
@pytest.mark.parametrize("xe,we", [(-118, 40), (-118, 0), (-126, 100), (-132, 60), (-142, 12), (-95, 0)])
@pytest.mark.parametrize("zeros", [False, True], ids=["full", "sparse"])
def test_activations_too_small_for_their_planes(layer, xe, we, zeros):
    """Activations whose lower bits lie under bf16's smallest subnormal, or that vanish in bf16 altogether, with weights that
    lift the sums out of there: as near to float64 as the fp32 instruction."""
    import torch
    x, w, bias = wl.make_tensors(layer, 2, 23)
    x = np.random.default_rng(7).standard_normal(x.shape, dtype=np.float32)
    if zeros:
        x[:, 4:8] = 0
    x, w, bias = np.ldexp(x, xe).astype(np.float32), np.ldexp(w, we).astype(np.float32), bias * 0
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = conv64(layer, x, zero_filled(wp, layer), bias)
    old = rel64(run(fp32_instruction(wp), xd, wp, bd, layer, relu=False), ref)
    vs = split_variants(wp)
    assert vs
    for v in vs:
        e = rel64(run(v, xd, wp, bd, layer, relu=False), ref)
        say(f"{layer.name} 2^{xe} * 2^{we} {nm.nm_variant_name(v)} {e:.3g} (fp32 instruction {old:.3g})")
        # one rounding per kept column, where the fp32 instruction has one per four: at most twice its distance
        assert e <= 2 * old + 1e-7, nm.nm_variant_name(v)


@pytest.mark.parametrize("layer", SMALL, ids=lambda l: l.name)
@pytest.mark.parametrize("xe,we", [(40, -118), (100, -126), (60, -142)])
def test_weights_too_small_for_their_planes(layer, xe, we):
    """A kept weight that three bf16 planes do not hold exactly keeps its layer off the three-plane kernel; one that was
    pruned does not."""
    import torch
    x, w, bias = wl.make_tensors(layer, 2, 29)
    x = np.ldexp(np.random.default_rng(8).standard_normal(x.shape, dtype=np.float32), xe).astype(np.float32)
    tiny, bias = np.ldexp(w, we).astype(np.float32), bias * 0
    wp = nm.nm_prune(tiny, layer.n, layer.m, layer.tile)
    assert not split_variants(wp)
    y = nm.nm_conv2d(torch.from_numpy(x).cuda(), wp, torch.from_numpy(bias).cuda(), layer.stride, layer.pad, layer.dil, False)
    torch.cuda.synchronize()
    assert rel64(y.cpu().numpy(), conv64(layer, x, zero_filled(wp, layer), bias)) <= 1e-6
    if layer.n < layer.m:
        mask = nm.nm_packed_mask(nm.nm_prune(w, layer.n, layer.m, layer.tile)).reshape(w.shape)
        assert split_variants(nm.nm_prune(np.where(mask, w, tiny), layer.n, layer.m, layer.tile))


def test_one_tiny_activation_among_ordinary_ones():
    """The other outputs stay what they are, bit for bit."""
    import torch
    layer = SMALL[0]
    x, w, bias = wl.make_tensors(layer, 2, 31)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
    bd = torch.from_numpy(bias).cuda()
    z = x.copy()
    x[0, 5, 5, 3], z[0, 5, 5, 3] = 1e-40, 0
    for v in split_variants(wp):
        a, b = (run(v, torch.from_numpy(t).cuda(), wp, bd, layer, relu=False) for t in (x, z))
        assert (a == b).all(), nm.nm_variant_name(v)


@pytest.mark.parametrize("n,m,cin", [(1, 4, 28), (2, 4, 16), (2, 4, 20), (1, 1, 8), (1, 1, 12), (4, 8, 16)])
@pytest.mark.parametrize("kind", ["uniform", "signed"])
@pytest.mark.parametrize("bias_on", [False, True])
def test_few_columns_no_further_from_float64(n, m, cin, kind, bias_on):
    import torch
    layer = L("few", 24, 24, cin, 64, 1, 1, 1, 0, 1, n, m, 16)
    x, w, bias = wl.make_tensors(layer, 4, 37)
    if kind == "signed":
        x = np.random.default_rng(3).standard_normal(x.shape, dtype=np.float32)
    bias = bias * np.float32(bias_on)
    wp = nm.nm_prune(w, n, m, 16)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = conv64(layer, x, zero_filled(wp, layer), bias)
    old = rel64(run(fp32_instruction(wp), xd, wp, bd, layer, relu=False), ref)
    for v in split_variants(wp):
        assert rel64(run(v, xd, wp, bd, layer, relu=False), ref) <= old, nm.nm_variant_name(v)


def test_fewest_columns_keep_the_fp32_instruction():
    """Up to six kept columns, of a whole layer or of one part of a K split, the planes' missing products weigh more than the
    roundings they save: the tuner leaves the three-plane forms out."""
    import torch
    for layer in (L("k1", 9, 9, 4, 64, 1, 1, 1, 0, 1, 1, 4, 16), L("k6", 9, 9, 12, 64, 1, 1, 1, 0, 1, 2, 4, 16),
                  L("k6d", 9, 9, 8, 64, 1, 1, 1, 0, 1, 6, 8, 16)):
        _, w, _ = wl.make_tensors(layer, 1, 41)
        wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
        assert split_variants(wp)
        say(layer.name)
        v, _ = nm.nm_autotune(nm.NM_F32, 1, 9, 9, layer.Cin, wp, True, 1, 0, 1, False)
        assert not nm.nm_variant_name(v).startswith("X3")
    nm.nm_cache_clear()


@pytest.mark.parametrize("tile,cout", [(1, 20), (5, 40), (4, 36), (12, 64), (32, 72), (16, 37)])
@pytest.mark.parametrize("n,m", [(2, 4), (1, 1)])
def test_outputs_computed_again_for_every_column_tile(tile, cout, n, m):
    """Outputs that are computed again, singly or four channels at a time, with residual, ReLU and a K split."""
    import torch
    layer = L("again", 11, 10, 68, cout, 3, 3, 1, 2, 2, n, m, tile)
    x, w, bias = wl.make_tensors(layer, 2, 43)
    x[0], bias = np.ldexp(x[0] - 0.5, -118), bias * 0
    x[1, 4, 5, 7], x[1, 9, 0, 60] = np.inf, -np.inf
    w = np.ldexp(w, 30).astype(np.float32)
    wp = nm.nm_prune(w, n, m, tile)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    for relu in (False, True):
        ref = run(fp32_instruction(wp), xd, wp, bd, layer, relu)
        rd = torch.from_numpy(np.random.default_rng(3).standard_normal(ref.shape, dtype=np.float32)).cuda()
        ref2 = run(fp32_instruction(wp), xd, wp, bd, layer, relu, rd)
        ok = np.isfinite(ref)
        assert ok[0].all() and not ok[1].all()
        for v in split_variants(wp):
            got = run(v, xd, wp, bd, layer, relu)
            assert rel64(got[0], ref[0].astype(np.float64)) <= 1e-6, nm.nm_variant_name(v)
            assert (np.isnan(got) == np.isnan(ref)).all() and (got[np.isinf(ref)] == ref[np.isinf(ref)]).all(), nm.nm_variant_name(v)
            assert rel64(got[ok], ref[ok].astype(np.float64)) <= 1e-6, nm.nm_variant_name(v)
            got = run(v, xd, wp, bd, layer, relu, rd)
            assert rel64(got[0], ref2[0].astype(np.float64)) <= 1e-6, nm.nm_variant_name(v)


@pytest.mark.parametrize("layer", [L("one_chunk", 20011, 1, 64, 200, 1, 1, 1, 0, 1, 2, 4, 16), L("three_chunks", 20011, 1, 192, 200, 1, 1, 1, 0, 1, 2, 4, 16),
                                   L("nine_chunks", 141, 142, 64, 136, 3, 3, 1, 1, 1, 2, 4, 16), L("two_chunks", 20011, 1, 68, 200, 1, 1, 1, 0, 1, 2, 4, 16),
                                   L("dense1", 20011, 1, 64, 200, 1, 1, 1, 0, 1, 1, 1, 16), L("dense3", 20011, 1, 136, 200, 1, 1, 1, 0, 1, 4, 8, 12)],
                         ids=lambda l: l.name)
def test_workgroups_walk_several_tiles(layer):
    """More output tiles than the chip holds workgroups, in numbers that do not divide evenly, with odd and even numbers of
    chunks a tile, ragged last tiles in both directions, with and without a residual: every form, every output."""
    import torch
    x, w, bias = wl.make_tensors(layer, 1, 47)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = conv64(layer, x, zero_filled(wp, layer), bias)
    res = np.random.default_rng(5).standard_normal(ref.shape, dtype=np.float32)
    rd = torch.from_numpy(res).cuda()
    vs = split_variants(wp)
    assert vs
    for v in vs:
        say(f"{layer.name} {nm.nm_variant_name(v)}")
        assert norm_err(run(v, xd, wp, bd, layer, relu=True), np.maximum(ref, 0)) <= FP32_TOL, nm.nm_variant_name(v)
        assert norm_err(run(v, xd, wp, bd, layer, relu=False, res=rd), ref + res) <= FP32_TOL, nm.nm_variant_name(v)


@pytest.mark.parametrize("cin,n,m", [(64, 2, 4), (192, 2, 4), (64, 1, 1)])
def test_small_activations_in_some_of_the_tiles_a_workgroup_walks(cin, n, m):
    """What the producers say about a tile is there when that tile is finished, one chunk a tile included."""
    import torch
    layer = L("late", 20011, 1, cin, 136, 1, 1, 1, 0, 1, n, m, 16)
    x, w, bias = wl.make_tensors(layer, 1, 53)
    small = np.zeros(20011, bool)
    small[[5, 64, 9000, 15003, 20010]] = True
    small[12345:12400] = True
    x[0, small], w, bias = np.ldexp(x[0, small] - 0.5, -128), np.ldexp(w, 60).astype(np.float32), bias * 0
    wp = nm.nm_prune(w, n, m, 16)
    xd, bd = torch.from_numpy(x).cuda(), torch.from_numpy(bias).cuda()
    ref = run(fp32_instruction(wp), xd, wp, bd, layer, False).astype(np.float64)[0, :, 0]
    for v in split_variants(wp):
        got = run(v, xd, wp, bd, layer, False)[0, :, 0]
        assert rel64(got[small], ref[small]) <= 1e-6, nm.nm_variant_name(v)
        assert rel64(got[~small], ref[~small]) <= 1e-6, nm.nm_variant_name(v)
