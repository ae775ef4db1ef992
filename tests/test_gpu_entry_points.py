"""The convolution's entry points against one another: the long forms with an argument for everything, and the block of arguments
that the binding passes, bit for bit on a call whose arguments all differ."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_2507_17301_amd import binding as nm
from gpu_util import FP32_TOL, say, norm_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_bias", [False, True])
@pytest.mark.parametrize("with_res", [False, True])
@pytest.mark.parametrize("relu", [0, 1])
def test_long_forms_and_the_block_of_arguments(with_bias, with_res, relu):
    import torch
    b, h, w, cin, cout, kh, kw = 3, 17, 26, 24, 40, 3, 2
    stride, pad, dil = (1, 2), (2, 1), (3, 4)
    rng = np.random.default_rng(6)
    x = rng.standard_normal((b, h, w, cin), dtype=np.float32)
    wt = rng.standard_normal((cout, kh, kw, cin), dtype=np.float32) * np.float32(0.1)
    bias = rng.standard_normal(cout, dtype=np.float32) if with_bias else None
    wz = oracle.prune(wt, 2, 4, 16)[2]
    ref = oracle.conv2d(x, wz, bias, stride, pad, dil, False)
    res = rng.standard_normal(ref.shape, dtype=np.float32) if with_res else None
    ref = ref + res if with_res else ref
    ref = np.maximum(ref, 0) if relu else ref
    wp = nm.nm_prune(wt, 2, 4, 16)
    xd = torch.from_numpy(x).cuda()
    bd = torch.from_numpy(bias).cuda() if with_bias else None
    rd = torch.from_numpy(res).cuda() if with_res else None
    say(f"entry points bias={with_bias} residual={with_res} relu={relu}")
    y = nm.nm_conv2d_res(xd, wp, rd, bd, stride, pad, dil, bool(relu))
    torch.cuda.synchronize()
    assert norm_err(y.cpu().numpy(), ref) <= FP32_TOL
    lib, ptr = nm.lib(), lambda t: None if t is None else t.data_ptr()
    geo = (*stride, *pad, *dil, relu)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)

    def call(entry, *tensors):
        out = torch.full_like(y, float("nan"))
        assert getattr(lib, entry)(xd.data_ptr(), nm.NM_F32, b, h, w, cin, wp.handle, *(ptr(t) for t in tensors), *geo,
                                   out.data_ptr(), nm.NM_F32, stream) == 0, entry
        torch.cuda.synchronize()
        return out

    assert torch.equal(call("nm_conv2d_res", bd, rd), y)
    assert torch.equal(call("nm_conv2d_static", bd, rd), y)
    if not with_res:
        assert torch.equal(call("nm_conv2d", bd), y)
