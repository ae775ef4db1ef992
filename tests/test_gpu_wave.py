"""The kernel for small fp32 layers (K axis dealt out over the wavefronts of a workgroup), every form forced, against
the CPU oracle: edges of its tiles, of its chunks and of the images, and values that unused operand slots must not see."""
import numpy as np
import pytest

import oracle
from paper_2507_17301_amd import binding as nm
from paper_2507_17301_amd import workloads as wl
from gpu_util import FP32_TOL, say, norm_err

pytestmark = pytest.mark.gpu

L = wl.ConvLayer

CASES = [
    # name, H, W, Cin, Cout, Kh, Kw, stride, pad, dil, n, m, tile | batch
    (L("kw_one_output", 1, 1, 4, 1, 1, 1, 1, 0, 1, 1, 1, 1), 1),                  # one pixel, one channel, four columns
    (L("kw_3x3", 7, 9, 64, 48, 3, 3, 1, 1, 1, 2, 4, 16), 1),                      # 63 pixels: the last block is ragged
    (L("kw_17_pixels", 17, 1, 64, 16, 1, 1, 1, 0, 1, 1, 1, 16), 1),
    (L("kw_cin48_T8", 9, 5, 48, 72, 3, 3, 1, 2, 2, 1, 4, 8), 2),                  # chunks end with the tap, half-empty row blocks
    (L("kw_cin100_s2", 11, 8, 100, 37, 3, 3, 2, 1, 1, 2, 4, 5), 1),               # odd channels out, images end inside a block
    (L("kw_T32_1x1", 5, 5, 96, 80, 1, 1, 1, 0, 1, 2, 8, 32), 3),
    (L("kw_1x1_s2", 9, 9, 128, 40, 1, 1, 2, 0, 1, 4, 8, 16), 1),
    (L("kw_deep", 7, 7, 512, 32, 3, 3, 1, 1, 1, 2, 4, 16), 1),                    # 72 chunks of 64, 144 of 32
    (L("kw_cin_groups", 6, 6, 64, 32, 3, 3, 1, 1, 1, 16, 64, 16), 1),             # uneven chunks: slots left over
    (L("kw_two_chunks", 4, 5, 1024, 16, 1, 1, 1, 0, 1, 1, 1, 16), 1),             # two, three and five chunks a wavefront,
    (L("kw_three_chunks", 5, 4, 128, 32, 3, 3, 2, 1, 1, 1, 1, 16), 3),            # all of a chunk kept, half, one column
    (L("kw_five_chunks", 5, 4, 256, 48, 3, 3, 1, 1, 1, 4, 8, 16), 1),
    (L("kw_five_sparse", 5, 4, 256, 48, 3, 3, 1, 1, 1, 1, 8, 32), 1),
    (L("kw_5x3_pad0", 8, 8, 20, 24, 5, 3, 1, 0, 1, 1, 4, 16), 1),
]


def _forms(wp):
    return [v for v in range(nm.nm_variant_count())
            if nm.nm_variant_name(v).startswith("KW_") and nm.nm_variant_legal(v, wp, nm.NM_F32, nm.NM_F32)]


def _forced(v, *a):
    import torch
    nm.nm_force_variant(v)
    try:
        y = nm.nm_conv2d_res(*a)
        torch.cuda.synchronize()
        assert nm.nm_last_variant() == v
    finally:
        nm.nm_force_variant(-1)
    return y.cpu().numpy()


@pytest.mark.parametrize("with_res", [False, True])
@pytest.mark.parametrize("layer,batch", CASES, ids=[c[0].name for c in CASES])
def test_every_form(layer, batch, with_res):
    import torch
    x, w, bias = wl.make_tensors(layer, batch, 17, weight_sigma=0.1)
    _, _, wz = oracle.prune(w, layer.n, layer.m, layer.tile)
    shape = (batch, layer.Ho, layer.Wo, layer.Cout)
    res = np.random.default_rng(3).standard_normal(shape).astype(np.float32) if with_res else None
    b = bias if with_res else None
    geo = (layer.stride, layer.pad, layer.dil, not with_res)
    ref = oracle.conv2d_res(x, wz, res, b, *geo) if with_res else oracle.conv2d(x, wz, b, *geo)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
    xd = torch.from_numpy(x).cuda()
    rd = torch.from_numpy(res).cuda() if with_res else None
    bd = torch.from_numpy(bias).cuda() if with_res else None
    forms = _forms(wp)
    assert len(forms) >= 4, "four shapes per chunk size"
    for v in forms:
        say(f"forced {nm.nm_variant_name(v)} on {layer.name} residual={with_res}")
        assert norm_err(_forced(v, xd, wp, rd, bd, *geo), ref) <= FP32_TOL, nm.nm_variant_name(v)


def test_values_of_columns_that_are_not_kept_stay_out():
    """Infinities and NaN in every column that some tile does not keep, in chunks with unused operand slots: an output
    is not finite only where the oracle's is not."""
    import torch
    layer = L("kw_inf", 6, 7, 40, 32, 3, 3, 1, 1, 1, 1, 4, 16)   # 10 of 40 channels kept; the second chunk of a tap fills 2 of 8 slots
    x, w, _ = wl.make_tensors(layer, 1, 5, weight_sigma=0.1)
    w[..., ::4] *= 10
    _, idx, _ = oracle.prune(w, 1, 4, 16)
    assert set((np.asarray(idx) % 40 % 4).ravel().tolist()) == {0}   # every fourth channel is kept, at every tap
    poison = [c for c in range(40) if c % 4]
    x[..., poison] = np.array([np.inf, -np.inf, np.nan], np.float32)[np.arange(len(poison)) % 3]
    x[0, 2, 3, 8] = np.nan                                           # and one value that is kept
    # (the oracle skips nothing that is kept: only the columns of a tile enter its sums)
    ref = np.zeros((1, 6, 7, 32), np.float32)
    xp = np.zeros((8, 9, 40), np.float64)
    xp[1:7, 1:8] = x[0]
    for j in range(2):
        kept = np.asarray(idx)[j].ravel()
        for co in range(16 * j, 16 * j + 16):
            wk = w[co].ravel()[kept].astype(np.float64)
            for h in range(6):
                for q in range(7):
                    ref[0, h, q, co] = xp[h:h + 3, q:q + 3].ravel()[kept] @ wk
    assert 0 < np.isnan(ref).sum() <= 9 * 32
    wp = nm.nm_prune(w, 1, 4, 16)
    for v in _forms(wp):
        say(f"forced {nm.nm_variant_name(v)} with infinities")
        y = _forced(v, torch.from_numpy(x).cuda(), wp, None, None, 1, 1, 1, False)
        ok = np.isfinite(ref)
        assert np.array_equal(np.isfinite(y), ok), nm.nm_variant_name(v)
        assert norm_err(y[ok], ref[ok]) <= FP32_TOL, nm.nm_variant_name(v)


# what the kernel gains grows with the K axis and falls with the blocks a CU gets: a layer on either side of each of the rule's
# lines (chunks of 32 channels at up to 256, 512, 768 and 1024 blocks, row blocks in pairs; dense layers beyond 512 blocks)
@pytest.mark.parametrize("layer,batch,wave", [
    (L("kd_1", 12, 26, 24, 16, 1, 1, 1, 0, 1, 2, 4, 16), 1, False), (L("kd_4", 14, 14, 128, 64, 1, 1, 1, 0, 1, 2, 4, 16), 2, True),
    (L("kd_7", 15, 36, 224, 128, 1, 1, 1, 0, 1, 1, 8, 16), 1, False), (L("kd_72", 14, 14, 256, 512, 3, 3, 1, 1, 1, 2, 4, 16), 1, True),
    (L("kd_pairs", 22, 32, 56, 48, 3, 3, 1, 1, 1, 4, 8, 16), 3, False), (L("kd_18", 23, 46, 64, 64, 3, 3, 2, 1, 1, 4, 8, 16), 10, False),
    (L("kd_3a_cu", 11, 11, 256, 256, 3, 3, 1, 1, 1, 2, 4, 16), 5, True), (L("kd_4a_cu", 61, 37, 16, 203, 3, 3, 2, 1, 1, 1, 4, 16), 2, False),
    (L("kd_dense", 5, 35, 504, 141, 1, 1, 1, 0, 1, 1, 1, 32), 7, False)], ids=lambda a: getattr(a, "name", None))
def test_untuned_default(layer, batch, wave):
    import torch
    x, w, bias = wl.make_tensors(layer, batch, 9, weight_sigma=0.1)
    _, _, wz = oracle.prune(w, layer.n, layer.m, layer.tile)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile)
    say(layer.name)
    y = nm.nm_conv2d(torch.from_numpy(x).cuda(), wp, torch.from_numpy(bias).cuda(), layer.stride, layer.pad, layer.dil, True)
    torch.cuda.synchronize()
    assert nm.nm_variant_name(nm.nm_last_variant()).startswith("KW_") == wave
    assert norm_err(y.cpu().numpy(), oracle.conv2d(x, wz, bias, layer.stride, layer.pad, layer.dil, True)) <= FP32_TOL
