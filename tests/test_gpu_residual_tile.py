"""The residual of the bf16 and fp8 convolutions, fetched in whole rows into the output tile: every form of the gather and
gather-free kernels on pixel and channel counts that end inside a tile, against the CPU oracle."""
import numpy as np
import pytest

import oracle
from paper_2507_17301_amd import binding as nm
from paper_2507_17301_amd import workloads as wl
from gpu_util import BF16_TOL, say, norm_err

pytestmark = pytest.mark.gpu

L = wl.ConvLayer

# pixels just over and under whole tiles, one chunk and several, output channels that end inside a 64- and a 128-wide tile
GRID = [(L("P1", 1, 1, 64, 64, 1, 1, 1, 0, 1, 2, 4, 16), 1), (L("P127_c72", 127, 1, 64, 72, 1, 1, 1, 0, 1, 2, 4, 16), 1),
        (L("P129_c136", 43, 3, 128, 136, 1, 1, 1, 0, 1, 2, 4, 16), 1), (L("P98_3x3", 7, 7, 64, 208, 3, 3, 1, 1, 1, 2, 4, 16), 2),
        (L("P33_T32", 11, 3, 256, 320, 1, 1, 1, 0, 1, 2, 8, 32), 1)]


@pytest.mark.parametrize("layer,batch", GRID, ids=[g[0].name for g in GRID])
@pytest.mark.parametrize("dtype", ["bf16", "f8"])
def test_residual_every_form(layer, batch, dtype):
    import torch
    dt, tdt = {"bf16": (nm.NM_BF16, torch.bfloat16), "f8": (nm.NM_F8E4M3, torch.float8_e4m3fn)}[dtype]
    x, w, bias = wl.make_tensors(layer, batch, 41, weight_sigma=0.1)
    wp = nm.nm_prune(w, layer.n, layer.m, layer.tile, dt)
    idx = nm.nm_packed_indices(wp).reshape(-1, layer.K // layer.m * layer.n)
    vals = nm.nm_packed_values(wp).reshape(*idx.shape, layer.tile)      # as stored: rounded to the handle's type
    wz = np.zeros((idx.shape[0] * layer.tile, layer.K), np.float32)
    for j in range(idx.shape[0]):
        for t in range(layer.tile):
            wz[j * layer.tile + t, idx[j]] = vals[j, :, t]
    wz = wz[:layer.Cout].reshape(w.shape)
    xd = torch.from_numpy(x).cuda().to(tdt)
    ref = oracle.conv2d(xd.float().cpu().numpy(), wz, bias, layer.stride, layer.pad, layer.dil, False)
    rd = torch.from_numpy(np.random.default_rng(2).standard_normal(ref.shape, dtype=np.float32)).cuda().to(torch.bfloat16)
    ref = np.maximum(ref + rd.float().cpu().numpy(), 0)
    bd = torch.from_numpy(bias).cuda()
    ran = 0
    try:
        for v in range(nm.nm_variant_count()):
            name = nm.nm_variant_name(v)
            if not name.startswith(("SP", "B16", "F8S", "F8W", "F8R")) or not nm.nm_variant_legal(v, wp, dt, nm.NM_BF16):
                continue
            say(f"{layer.name} {dtype} {name}")
            nm.nm_force_variant(v)
            y = nm.nm_conv2d_res(xd, wp, rd, bd, layer.stride, layer.pad, layer.dil, True)
            torch.cuda.synchronize()
            assert norm_err(y.float().cpu().numpy(), ref) <= BF16_TOL, name
            ran += 1
    finally:
        nm.nm_force_variant(-1)
    assert ran
